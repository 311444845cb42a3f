// eql_launch_impl.h -- tile choice and launches for one group order and element
// type.  Included only by eql_inst.hip, which is compiled once per (T, dtype).
#pragma once
#include "eql_gemm.h"
#include "eql_kernels.h"
#include "eql_wgrad.h"
#include "eql_wgrad_rd.h"
#include "eql_bwd_fused.h"
#include "eql_launch.h"
#include "eql_xs.h"

namespace eqk {

template <int T, int DT>
hipError_t wspec_t(const void* w, void* wspec, int Cin, int Cout, hipStream_t s) {
  const WspecDims d = wspec_dims(Cin, Cout);
  const int omax = d.CoF > d.CoutB ? d.CoF : d.CoutB;  // tiles cover both layouts
  const int cmax = d.CiF > d.CinB ? d.CiF : d.CinB;
  constexpr int WO = 256 * (DT != kF32 ? 8 : 4) / kWsC;  // output channels per tile (eql_wspec_kernel)
  hipLaunchKernelGGL((eql_wspec_kernel<T, DT>),
                     dim3((unsigned)((omax + WO - 1) / WO), (unsigned)((cmax + kWsC - 1) / kWsC)),
                     dim3(256), 0, s, w, wspec, Cin, Cout, d.CoF, d.CiF, d.CinB, d.CoutB);
  return hipGetLastError();
}

template <int T, int DT, bool BWD, int RT, bool ODD, bool GATHER, int FORM>
hipError_t xs_variant(const GemmArgs& a) {
  auto k = eql_xs_kernel<T, DT, BWD, RT, ODD, GATHER, FORM>;
  const XsPlan& p = a.plan;
  const bool w16 = DT != kF32;
  const int nksw = a.Ci_pad / xs_kf_c(w16), w_tiles = a.Co_pad / 16, n_ot = (a.Co + 15) / 16;
  // the kernel's assumptions: whole padded blocks, the spectrum of RT row
  // tiles and the bias in LDS, rows of a workgroup below 2^31 bytes
  if (p.nks != xs_nks(a.Ci, w16) || p.nks > nksw || a.Ci_pad % 32 != 0 || n_ot > w_tiles || p.osplit < 1 ||
      p.osplit > n_ot || p.NW < 1 || p.NW > 8 || p.lds_bytes > kLdsBytes || p.kc < 1 ||
      FORM != p.form || (FORM != kXsPipe && (FORM == kXsChunk) != (p.kc < p.nks)) ||
      (FORM == kXsChunk && (p.kc % 2 != 0 || (n_ot + p.osplit - 1) / p.osplit > p.NW)) ||
      (FORM == kXsPipe && (p.osplit != 1 || n_ot >= p.NW ||
                           16 * RT * p.kc * (xs_kf_c(w16) / 4) > xs_pipe_units(T) * 64 * (p.NW - n_ot))) ||
      p.lds_bytes < (FORM == kXsPipe ? 2 : 1) * RT * p.kc * T * 1024 + (BWD ? 0 : ((n_ot + p.osplit - 1) / p.osplit) * 64))
    return hipErrorInvalidValue;
  if (p.lds_bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds_bytes);
    if (e != hipSuccess) return e;
  }
  const int64_t groups = (a.N + 16 * RT - 1) / (16 * RT);
  if constexpr (FORM == kXsPipe) {  // one workgroup a CU, which walks its row groups
    const int64_t cus = device_cu_count();
    hipLaunchKernelGGL(k, dim3((unsigned)(groups < cus ? groups : cus)), dim3(64 * p.NW), p.lds_bytes, a.stream, a.in,
                       a.wsp, a.bias, a.out, a.N, (int64_t)0, a.Ci, a.Co, p.nks, nksw, p.kc, n_ot, 1, w_tiles, a.geo);
    return hipGetLastError();
  }
  const int64_t most = launch_blocks(64 * p.NW) / p.osplit / 8 * 8;  // row groups of one launch
  for (int64_t g0 = 0; g0 < groups; g0 += most) {
    const int64_t n = groups - g0 < most ? groups - g0 : most;
    hipLaunchKernelGGL(k, dim3((unsigned)((n + 7) / 8 * 8 * p.osplit)), dim3(64 * p.NW), p.lds_bytes, a.stream, a.in,
                       a.wsp, a.bias, a.out, a.N, g0 * 16 * RT, a.Ci, a.Co, p.nks, nksw, p.kc, n_ot, p.osplit,
                       w_tiles, a.geo);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int T, int DT, bool BWD, bool GATHER = false>
hipError_t xs_t(const GemmArgs& a) {
  hipError_t r = hipErrorInvalidValue;
  static_for<3>([&](auto ri) {
    constexpr int RT = 1 << decltype(ri)::value;
    constexpr bool pipe = xs_pipe_inst(T, DT != kF32, RT) && !GATHER;
    if (a.plan.RT != RT) return;
    if constexpr (pipe) {
      if (a.plan.form == kXsPipe) {
        r = xs_variant<T, DT, BWD, RT, false, false, kXsPipe>(a);
        return;
      }
    }
    if constexpr (xs_rt_inst(T, RT)) {
      if constexpr (DT != kF32 && T % 2 == 1 && !GATHER) {
        if (a.Ci % 2 != 0) {
          r = a.plan.form == kXsChunk ? xs_variant<T, DT, BWD, RT, true, false, kXsChunk>(a)
                                      : xs_variant<T, DT, BWD, RT, true, false, kXsWhole>(a);
          return;
        }
      }
      r = a.plan.form == kXsChunk ? xs_variant<T, DT, BWD, RT, false, GATHER, kXsChunk>(a)
                                  : xs_variant<T, DT, BWD, RT, false, GATHER, kXsWhole>(a);
    }
  });
  return r;
}

// Forward with the implicit patch gather (group convolution, T in {1, 2, 4}).
template <int T, int DT>
hipError_t gemm_gather_t(const GemmArgs& a) {
  if constexpr (T == 1 || T == 2 || T == 4) return xs_t<T, DT, false, true>(a);
  return hipErrorInvalidValue;
}

// The split-partial reduction (both weight-gradient kernels write the same
// partial layout).
template <int T, int DT>
hipError_t wgrad_reduce(const WgradArgs& a, const WgradPlan& p);

template <int T, int DT, int CT, int OT>
hipError_t wgrad_rd_variant(const WgradArgs& a, const WgradPlan& p) {
  if (p.S > 0) {
    constexpr int NW = kRdWaves;
    const int lds = (NW - 1) * rd_wave_acc_bytes<T, CT, OT>() + NW * OT * 16 * 4;
    auto k = eql_wgrad_rd_kernel<T, DT, CT, OT, NW>;
    if (lds > kLdsBytes) return hipErrorInvalidValue;
    if (lds > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
    }
    const int64_t G = (int64_t)p.S * p.n_ct * p.n_ot;
    const int64_t blocks = (G + 7) / 8 * 8;  // whole groups of 8 (one per XCD)
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(64 * NW), lds, a.stream, a.x, a.dy, a.part,
                       a.db ? a.dbpart : nullptr, a.N, a.Cin, a.Cout, p.rows_per_split, p.n_ct,
                       p.n_ot, p.S, p.Cin_pad, p.Cout_pad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return wgrad_reduce<T, DT>(a, p);
}

template <int T, int DT, int WGC, int CT, int OTW>
hipError_t wgrad_variant(const WgradArgs& a, const WgradPlan& p) {
  if (p.S > 0) {
    // whole groups of 8 splits (see the tile order in eql_wgrad_kernel)
    const int64_t n_blocks = (int64_t)(p.S + 7) / 8 * 8 * p.n_ct * p.n_ot;
    hipLaunchKernelGGL((eql_wgrad_kernel<T, DT, WGC, 8 / WGC, CT, OTW>), dim3((unsigned)n_blocks),
                       dim3(512), 0, a.stream, a.x, a.dy, a.part, a.db ? a.dbpart : nullptr, a.N,
                       a.Cin, a.Cout, p.rows_per_split, p.n_ct, p.n_ot, p.S, p.Cin_pad,
                       p.Cout_pad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return wgrad_reduce<T, DT>(a, p);
}

template <int T, int DT>
hipError_t wgrad_reduce(const WgradArgs& a, const WgradPlan& p) {
  // threads, items per workgroup and split groups of eql_wgrad_reduce_kernel
  const int64_t items = (int64_t)(p.Cin_pad / 4) * p.Cout_pad;
  int nthr = 0, ipw = 0, G = 0;
  wgrad_reduce_shape(T, p.S, items, nthr, ipw, G);
  const int NS = nthr / G;
  const unsigned blocks =
      (unsigned)((items + ipw - 1) / ipw + (a.db ? (a.Cout + NS - 1) / NS : 0));
  if (nthr == 256)
    hipLaunchKernelGGL((eql_wgrad_reduce_kernel<T, DT, 256>), dim3(blocks), dim3(256), 0, a.stream,
                       a.part, a.dbpart, a.dw, a.db, p.S, a.Cin, a.Cout, p.Cin_pad, p.Cout_pad, ipw, G);
  else
    hipLaunchKernelGGL((eql_wgrad_reduce_kernel<T, DT, 1024>), dim3(blocks), dim3(1024), 0, a.stream,
                       a.part, a.dbpart, a.dw, a.db, p.S, a.Cin, a.Cout, p.Cin_pad, p.Cout_pad, ipw, G);
  return hipGetLastError();
}

// Single-pass backward: the fused kernel (one workgroup per row split), then
// the split-partial reduction of the weight gradient.
template <int T, int DT, int WGC, int CT, int OTW>
hipError_t fused_variant(const FusedArgs& f, const FusedPlan& p) {
  constexpr int BC = WGC * 16 * CT, BO = (8 / WGC) * 16 * OTW;
  constexpr int KR = DT != kF32 ? 32 : 16;
  if (p.BC != BC || p.BO != BO || p.KR != KR || p.nks * KR > BO || p.C16 > BC ||
      p.lds != fused_lds_bytes(T, BC, BO, KR, p.nks, p.C16, p.dbuf != 0) || p.lds > kLdsBytes)
    return hipErrorInvalidValue;
  WgradArgs a{};
  a.x = f.x;
  a.dy = f.dy;
  a.dw = f.dw;
  a.db = f.db;
  a.part = f.part;
  a.dbpart = f.dbpart;
  a.N = f.N;
  a.Cin = f.Cin;
  a.Cout = f.Cout;
  a.stream = f.stream;
  WgradPlan wp{};
  wp.S = p.S;
  wp.Cin_pad = BC;
  wp.Cout_pad = BO;
  if (p.S > 0) {
    auto k = eql_bwd_fused_kernel<T, DT, WGC, CT, OTW>;
    if (p.lds > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)p.S), dim3(512), p.lds, f.stream, f.x, f.dy, f.wsp, f.dx, f.part,
                       f.db ? f.dbpart : nullptr, f.N, f.Cin, f.Cout, p.rows_per_split, p.S, f.CinB,
                       f.CoutB, p.nks, p.dbuf);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return wgrad_reduce<T, DT>(a, wp);
}

template <int T, int DT>
hipError_t fused_t(const FusedArgs& f, const FusedPlan& p) {
  // the variants of fused_plan that fit the registers (fused_variant_ok)
#define EQK_FU(W_, C_, O_)                                                  \
  if constexpr (DT != kBF16 && fused_variant_ok(T, DT == kF16, W_, C_, O_)) { \
    if (p.wgc == (W_) && p.ct == (C_) && p.otw == (O_))                    \
      return fused_variant<T, DT, W_, C_, O_>(f, p);                       \
  }
  EQK_FU(2, 1, 1)
  EQK_FU(4, 1, 1)
  EQK_FU(2, 1, 2)
  EQK_FU(2, 2, 1)
  EQK_FU(2, 1, 3)
#undef EQK_FU
  return hipErrorInvalidValue;
}

template <int T, int DT>
hipError_t wgrad_t(const WgradArgs& a, const WgradPlan& p) {
  // large-tile plan: its pre-passes and product kernel ran (launch_wgrad_big)
  if (p.kind == 2) return wgrad_reduce<T, DT>(a, p);
  if (p.kind == 1) {
#define EQK_RD(C_, O_)                                             \
  if constexpr (rd_fits(T, C_, O_)) {                              \
    if (p.ct == (C_) && p.otw == (O_)) return wgrad_rd_variant<T, DT, C_, O_>(a, p); \
  }
    EQK_RD(1, 1)
    EQK_RD(1, 2)
    EQK_RD(2, 1)
    EQK_RD(2, 2)
    EQK_RD(2, 4)
    EQK_RD(4, 2)
#undef EQK_RD
    return hipErrorInvalidValue;
  }
  // the variants of wgrad_plan whose accumulators fit (CT * OTW * T * 4 <= 96)
#define EQK_WG(W_, C_, O_)                                                                    \
  if constexpr ((C_) * (O_) * T * 4 <= 96 &&                                                 \
                T * ((W_) * 16 * (C_) + (8 / (W_)) * 16 * (O_)) * 64 <= 160 * 1024 - 4096) {   \
    if (p.wgc == (W_) && p.ct == (C_) && p.otw == (O_))                                      \
      return wgrad_variant<T, DT, W_, C_, O_>(a, p);                                         \
  }
  EQK_WG(2, 1, 1)
  EQK_WG(2, 2, 1)
  EQK_WG(2, 3, 1)
  EQK_WG(2, 1, 2)
  EQK_WG(2, 1, 3)
  EQK_WG(4, 1, 1)
  EQK_WG(4, 1, 2)
  EQK_WG(4, 1, 3)
#undef EQK_WG
  return hipErrorInvalidValue;
}

}  // namespace eqk

// eql_launch.h -- internal launch interface between the C-ABI layer and the
// per-dtype kernel instantiation units.  Host code only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "eql_config.h"

namespace eqk {

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

constexpr int kLdsBytes = 160 * 1024;
// Workgroups of one launch: HIP refuses 2^32 threads and more, so a pass over
// more rows than that takes several launches.
constexpr int64_t launch_blocks(int threads) { return (((int64_t)1 << 32) - 1) / threads; }

// Padded extents of the weight spectrum: rows and contraction channels to 32
// (whole tiles of 16 rows, whole steps).
constexpr int kColPad = 32;
struct WspecDims {
  int CoF, CiF, CinB, CoutB;
};
inline WspecDims wspec_dims(int Cin, int Cout) {
  const int ci = round_up(Cin, kColPad), co = round_up(Cout, kColPad);
  return {co, ci, ci, co};
}

// Plan of eql_xs_kernel for Ci -> Co over N rows: row tiles per workgroup,
// waves, output splits, steps, steps staged at once (all of them, an even chunk
// with at most NW output tiles per split, or, pipelined, any chunk with fewer
// output tiles than waves) and the LDS.
enum XsForm { kXsWhole = 0, kXsChunk = 1, kXsPipe = 2 };
struct XsPlan {
  int RT, NW, osplit, nks, kc, lds_bytes;
  int form;  // XsForm
};
constexpr int xs_kf_c(bool w16) { return w16 ? 32 : 16; }  // contraction channels per step
inline int xs_nks(int Ci, bool w16) { return (Ci + xs_kf_c(w16) - 1) / xs_kf_c(w16); }
// row tiles that have an instantiation
constexpr bool xs_rt_inst(int T, int RT) { return RT == 1 || (RT == 2 && T <= 8) || (RT == 4 && T <= 4); }
// the pipelined form: its instantiations, and the units of 4 channels a staging
// thread holds (64 raw words)
constexpr bool xs_pipe_inst(int T, bool w16, int RT) { return w16 && T == 8 && RT == 4; }
constexpr int xs_pipe_units(int T) { return 64 / (2 * T); }
XsPlan xs_plan(int64_t N, int T, int Ci, int Co, int dt, int cus);

// Compute units of the current device (cached); 256 if unknown.
int device_cu_count();

// Plan of the split-row weight gradient: kernel, workgroup tile, split count
// and the padded partial extents.  kind 0: eql_wgrad_kernel (operands staged
// in LDS, a WGC x WGO wave grid of CT x OTW blocks of 16 x 16 channels per
// wave); kind 1: eql_wgrad_rd_kernel (register-direct operands, kRdWaves
// waves on one tile of CT x OTW blocks).  Depends only on the problem, not on
// the device, so results are reproducible across devices of the same model.
constexpr int kRdWaves = 4;
// Register-direct variants whose accumulators and two raw chunk buffers fit
// one wave per SIMD: 4T (CT*OT + 2 (CT + OT)) <= 400 registers.
constexpr bool rd_fits(int T, int CT, int OT) { return 4 * T * (CT * OT + 2 * (CT + OT)) <= 400; }
struct WgradPlan {
  int kind;
  int wgc, ct, otw; // variant: wave grid rows (WGO = 8 / wgc), tiles per wave
  int BC, BO;       // channel tile of one workgroup
  int KR;           // rows per chunk
  int n_ct, n_ot;   // channel tiles
  int S;            // splits
  int64_t rows_per_split;
  int Cin_pad, Cout_pad;
  size_t part_bytes, dbpart_bytes;
  // kind 2 (eql_wgrad_big.h): row-contiguous spectra of x and dy in the
  // workspace, N_pad rows (a multiple of 64) per plane row
  int64_t N_pad;
  size_t xs_bytes, ds_bytes;
};
// dt: element type code.  Plans whose workspace would exceed max_ws fall
// back to the split-row kernels (the allocation-free entry point passes its
// static scratch size).
WgradPlan wgrad_plan(int64_t N, int T, int Cin, int Cout, int dt, size_t max_ws = (size_t)-1);
inline size_t align256z(size_t v) { return (v + 255) / 256 * 256; }
// workspace of a plan: partials, bias partials, then (kind 2) the spectra
inline size_t wgrad_workspace(const WgradPlan& p) {
  return align256z(p.part_bytes) + align256z(p.dbpart_bytes) + align256z(p.xs_bytes) + align256z(p.ds_bytes);
}
// Three-product complex bins in the large-tile kernels (fp32, T = 4;
// 96-channel output tiles).  EQL_GAUSS=0 takes the four-product form
// everywhere, =1 the three-product one everywhere; unset, the forward and
// input gradient take three products and the weight gradient as below.
int gauss_forced();  // -1 unset, 0, 1
inline bool big_gauss(int T, int dt) { return T == 4 && dt == kF32 && gauss_forced() != 0; }

// Large-tile weight gradient (kind 2): T in {2, 4}, and the spectra of x and
// dy addressable with 31-bit offsets.  Taken by default from
// wgrad_big_min_c channels each way, where it measured faster than the
// register-direct kernel (T = 4, 32,768 rows, weight and bias gradient, µs
// large-tile / register-direct: fp16 463 / 864 at c = 768, 261 / 221 at 512;
// fp32 2059 / 3592 at 768, 988 / 888 at 512; bf16 261 / 320 at 512, 109 / 88
// at 256);
// EQL_WGRAD_KIND=2 forces it where it fits.  fp32 at T = 4 takes the
// three-product complex bin with 96-channel o-tiles (big_gauss) where the
// 128-channel tiles alone fill the 256 CUs (c = 2048: 12.04 against 12.71
// ms); with fewer tiles the row splits balance the four-product tiles as
// well and the three products measured 2% slower (c = 1024: 3.48 vs 3.41 ms).
inline int wgrad_big_min_c(int dt) { return dt == kBF16 ? 512 : 768; }
inline int wgrad_big_o_tile(int T, int Cin, int Cout, int dt) {
  if (T != 4 || dt != kF32) return 128;
  const int f = gauss_forced();
  const int64_t tiles128 = (int64_t)((Cin + 127) / 128) * ((Cout + 127) / 128);
  return f == 1 || (f < 0 && tiles128 >= 256) ? 96 : 128;
}
// Rows of the row-contiguous spectra: N in whole 64-row blocks of the
// pre-pass, plus one more block where that count is even, so that the channel
// rows' pitch is an odd multiple of 128 bytes (16-bit) or twice one (fp32)
// and the rows one step reads spread over the L2 sets instead of sharing a
// few (a pitch of 32,768 rows is 64 KB).  The extra rows are zero.
inline int64_t wgrad_big_npad(int64_t N) {
  const int64_t blocks = (N + 63) / 64;
  return (blocks % 2 == 0 ? blocks + 1 : blocks) * 64;
}
inline bool wgrad_big_fits(int64_t N, int T, int Cin, int Cout, int dt) {
  const int64_t eb = dt == kF32 ? 4 : 2;
  const int64_t np = wgrad_big_npad(N);
  const int64_t bo = wgrad_big_o_tile(T, Cin, Cout, dt);
  const int64_t ci = (Cin + 127) / 128 * 128, co = (Cout + bo - 1) / bo * bo;
  const int64_t lim = (int64_t)1 << 31;
  return (dt == kF32 || dt == kF16 || dt == kBF16) && (T == 2 || T == 4) && N > 0 && (int64_t)T * ci * np * eb < lim &&
         (int64_t)T * co * np * eb < lim && (int64_t)64 * (Cin > Cout ? Cin : Cout) * T * eb < lim;
}

// Shape of the partial reduction: NTHR threads per workgroup, runs of IPW
// items (IPW * 16 bytes per split and plane), G = NTHR / (IPW * T) split
// groups (at most 32).  Up to 64 splits: 256 threads and IPW = min(16, 64/T)
// (the headline's 40 splits: 8 items x 4 groups, 10 splits per thread in two
// batches; 10.8 us against 12.1 us with 1024 threads); more splits: 1024
// threads and IPW = 16 where that still gives 128 workgroups, else 8 or 4
// (16-item runs measured as fast as or faster than 4..64).
// EQL_RED_IPW forces IPW (A/B timing).
inline void wgrad_reduce_shape(int T, int S, int64_t items, int& nthr, int& ipw, int& G) {
  int forced = 0;
  if (const char* e = getenv("EQL_RED_IPW")) forced = atoi(e);
  nthr = S <= 64 ? 256 : 1024;
  if ((forced == 4 || forced == 8 || forced == 16 || forced == 32 || forced == 64) && forced * T <= nthr) {
    ipw = forced;
  } else if (nthr == 256) {
    ipw = 64 / T < 1 ? 1 : (64 / T > 16 ? 16 : 64 / T);
  } else {
    for (ipw = 16; ipw > 4; ipw /= 2)
      if ((items + ipw - 1) / ipw >= 128) break;
  }
  G = nthr / (ipw * T);
  if (G > 32) G = 32;
}

// Plan of the single-pass backward (eql_bwd_fused_kernel): the variant (wave
// grid rows, c-tiles, o-tiles per wave of the eql_wgrad_kernel grid) whose
// workgroup tile BC x BO holds every channel pair of the layer, the row
// splits, the input-gradient steps of KR output channels, and the LDS.  ok = 0
// when the layer does not take this path (then eqlinear_backward runs the
// input- and weight-gradient kernels one after the other).  Depends only on
// the problem, not on the device.
struct FusedPlan {
  int ok;
  int wgc, ct, otw, BC, BO;
  int KR, nks, C16;  // rows per chunk (= output channels per step), steps, Cin rounded to 16
  int dbuf, lds;     // two staging buffers; dynamic LDS bytes
  int S;
  int64_t rows_per_split;
  size_t part_bytes, dbpart_bytes;
};
FusedPlan fused_plan(int64_t N, int T, int Cin, int Cout, int dt);  // none for bf16
// Variants of eql_bwd_fused_kernel built for group order T and element
// type (fp16 or fp32): those that fit the 256 registers of a lane at two waves per SIMD
// without spilling (the weight-gradient accumulators, the input-gradient
// tile, two chunks of prefetched raw rows and the transforms; found by
// compiling every variant, and the post-build check refuses a spilling one).
constexpr bool fused_variant_ok(int T, bool f16, int ct, int otw) {
  const int tmax = (ct == 1 && otw == 1) ? (f16 ? 6 : 11)
                   : (ct == 2 && otw == 1) ? (f16 ? 5 : 7)
                   : (ct == 1 && otw == 2) ? (f16 ? 4 : 5)
                   : (ct == 1 && otw == 3) ? (f16 ? 2 : 3)
                                           : 0;
  return T <= tmax;
}
// 4 x 1 waves with one 16-channel block each: fewer registers than 2 x 4
constexpr bool fused_variant_ok(int T, bool f16, int wgc, int ct, int otw) {
  return wgc == 4 && ct == 1 && otw == 1 ? T <= (f16 ? 8 : 11) : fused_variant_ok(T, f16, ct, otw);
}
// LDS bytes of one workgroup of eql_bwd_fused_kernel: one or two staging
// buffers (x planes, dy planes by row, dy planes by output channel), then the
// weight spectrum.  Every staged row is 64 bytes: KR rows (weight-gradient
// staging) or KR output channels (input-gradient staging and weights) of one
// element each.
constexpr int kFusedRowBytes = 64;
inline int fused_lds_bytes(int T, int BC, int BO, int KR, int nks, int C16, bool dbuf) {
  const int stg = T * (BC + BO) * kFusedRowBytes + nks * T * KR * kFusedRowBytes;
  return (dbuf ? 2 : 1) * stg + nks * T * C16 * kFusedRowBytes;
}

struct GemmArgs {
  const void* in;
  const void* wsp;   // plane block of the layout this pass reads
  const void* bias;  // forward only; may be null
  void* out;
  int64_t N;
  int Ci, Co, Ci_pad;
  int Co_pad;        // padded rows of the weights this pass reads
  XsPlan plan;
  hipStream_t stream;
  GatherGeom geo;    // implicit patch gather only (else zero)
};

struct WgradArgs {
  const void* x;
  const void* dy;
  void* dw;
  void* db;          // may be null
  float* part;
  float* dbpart;
  void* xs;          // kind 2: row-contiguous spectra of x and dy
  void* ds;
  int64_t N;
  int Cin, Cout;
  hipStream_t stream;
};

struct FusedArgs {
  const void* x;
  const void* dy;
  const void* wsp;   // backward-layout plane block of the weight spectrum
  void* dx;
  void* dw;
  void* db;          // may be null
  float* part;
  float* dbpart;
  int64_t N;
  int Cin, Cout, CinB, CoutB;
  hipStream_t stream;
};

// Launches of one group order and element type (eql_inst.hip, one object per
// (T, dtype) so the instantiations build in parallel).
template <int T, int DT>
struct Inst {
  static hipError_t wspec(const void* w, void* wspec, int Cin, int Cout, hipStream_t s);
  static hipError_t gemm(bool bwd, const GemmArgs& a);
  static hipError_t gemm_gather(const GemmArgs& a);
  static hipError_t wgrad(const WgradArgs& a, const WgradPlan& p);
  static hipError_t bwd_fused(const FusedArgs& a, const FusedPlan& p);
};

// Dispatch over T and the element type code dt (eql_dispatch.cpp).
hipError_t launch_wspec(int dt, int T, const void* w, void* wspec, int Cin, int Cout, hipStream_t s);
hipError_t launch_gemm(int dt, int T, bool bwd, const GemmArgs& a);

// Large-tile forward / input gradient (eql_gemm_big.h): T in {2, 4},
// contraction channels a multiple of 32, and every 128-row tile of the input
// and output below 2^31 bytes.  Taken by default for wide layers (both
// channel counts at least kBigMinC), where the spectral products bound the
// pass.  Against eql_xs_kernel (us, eql_xs_kernel / large tiles, forward, inputs
// from HBM) the line is right at T = 4 for many rows and 512 channels or more
// (fp16 1024 x 1024, 32,768 rows 566 / 435; 4,096 rows 84 / 58; 512 x 512, 8,192
// rows 47 / 35; bf16 1024 x 1024, 32,768 rows 592 / 487), level at 256 x 256 in 16
// bits (44 / 46 at 32,768 rows), and wrong where the tiles cannot fill the device
// or the spectrum is small: few rows (fp16 1024 x 1024, 512 rows 16 / 47; fp32
// 256 x 256, 512 rows 12 / 73), 256 x 1024 (fp16, 32,768 rows 129 / 168), fp32 at
// 256 channels (32,768 rows 207 / 231) and T = 2 up to 1024 channels (fp16 1024 x
// 1024, 32,768 rows 230 / 313).  EQL_GEMM_BIG=0 never takes it, =1 whenever the shape
// allows (tests, A/B timing).
struct BigArgs {
  const void* in;
  const void* wsp;   // plane block of the layout this pass reads
  const void* bias;  // forward only; may be null
  void* out;
  int64_t N;
  int Ci, Co;        // contraction and output channels of this pass
  int w_rows, w_pitch;  // padded rows (>= Co) and contraction channels (>= Ci) of the spectrum
  hipStream_t stream;
};
constexpr int kBigMinC = 256;
int gemm_big_forced();  // -1 unset, 0, 1

inline bool gemm_big_fits(int T, int Ci, int Co, int dt) {
  const int64_t eb = dt == kF32 ? 4 : 2;
  return (dt == kF32 || dt == kF16 || dt == kBF16) && (T == 2 || T == 4) && Ci % 32 == 0 && Co >= 1 &&
         (int64_t)128 * Ci * T * eb < ((int64_t)1 << 31) && (int64_t)128 * Co * T * eb < ((int64_t)1 << 31);
}
inline bool gemm_big_choose(int T, int Ci, int Co, int dt) {
  if (!gemm_big_fits(T, Ci, Co, dt)) return false;
  const int f = gemm_big_forced();
  if (f >= 0) return f == 1;
  return Ci >= kBigMinC && Co >= kBigMinC;
}
hipError_t launch_gemm_big(int dt, int T, bool bwd, const BigArgs& a);
hipError_t launch_gemm_gather(int dt, int T, const GemmArgs& a);
hipError_t launch_wgrad(int dt, int T, const WgradArgs& a, const WgradPlan& p);
// kind 2: the spectrum pre-passes and the product kernel (launch_wgrad then
// runs the reduction)
hipError_t launch_wgrad_big(int dt, int T, const WgradArgs& a, const WgradPlan& p);
hipError_t launch_bwd_fused(int dt, int T, const FusedArgs& a, const FusedPlan& p);

// Encoder block kernels (eql_block.h): a layer-norm row of whole 16-byte
// vectors, at most four a lane of a 256-thread workgroup; attention over at
// most 256 tokens (the scores of a query tile stay in registers, K and V^T of a
// head in LDS).
constexpr int kNormMaxBytes = 4 * 256 * 16;
constexpr int kAttnMaxL = 256;
hipError_t launch_group_norm(int dt, const void* x, const void* w, const void* b, void* y, int64_t rows, int T, int C,
                             float eps, int cus, hipStream_t stream);
hipError_t launch_attention(int dt, const void* qkv, void* o, int64_t B, int L, int H, int D, float scale, int cus,
                            hipStream_t stream);

}  // namespace eqk

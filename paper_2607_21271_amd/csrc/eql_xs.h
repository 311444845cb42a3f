// eql_xs.h -- forward and input-gradient kernel of the C_T equivariant linear
// layer for gfx950 with the activation spectrum stationary in LDS: rDFT of the
// activations -> per-bin MFMA products -> irDFT (+ bias), fused in one pass
// over the rows (Alg. 1 steps 1-4; Sec. 3.5).
//
// Work split.  A workgroup takes 16 * RT rows and a run of output tiles of 16
// channels.  It transforms its rows once over all contraction channels and
// keeps their T planes in LDS as complete MFMA operands; after one barrier its
// waves never meet again: each takes every NW-th output tile, reads that
// tile's weights straight from global memory into registers (one step ahead of
// the products) and the row operands from LDS, and runs the inverse transform
// and the stores on its own.
//
// Fragment order.  An operand fragment (16 rows or output channels x KF
// contraction channels of one plane, 16 bytes a lane) is one block of 1 KB in
// lane order: lane (g, i) holds row i, contraction channels KWM * g .. of the
// step.  The weight spectrum is stored as such blocks, [tile][step][plane], so
// a wave's weights are one contiguous stream that needs no LDS, no swizzle and
// no barrier.  In LDS the lane slot is permuted by the step (xs_slot) so that
// the units of one row, which the staging writes together, fall on different
// banks.
//
// Few workgroups fill a CU and each stages its rows at once; where the
// spectrum of all channels is too large for that, chunks of kc steps are
// staged in turn and the tiles' accumulators stay in registers (kXsChunk).
//
// Pipelined form (kXsPipe, T = 8, 16-bit, five or six output tiles).  Chunks leave
// the products idle while a chunk is staged, and two splits stage every row twice.
// Here a workgroup a CU walks groups of 64 rows; some waves only stage, into
// one of two LDS buffers, the others run the products of the chunk before from
// the other.  A wave's memory counter retires loads in order, so rows prefetched
// by the wave that streams the weights would be waited for with the next weights;
// a staging wave's loads are its own, and the next chunk's are in flight across
// the barrier.  Four row tiles a weight fragment: with two the pipelined form is level
// with the barrier-per-step kernel (36.6 us below); loading the weights further
// ahead changed nothing.  384 -> 96, 12,608 rows, inputs from HBM (floor 19 us),
// barrier-per-step kernel / chunks / this form: fp16 36.7 / 39.5 / 29.9, bf16
// 37.5 / 41.6 / 34.2.
//
// What bounds it, and why this form.  A kernel that met at a barrier every
// contraction step, staged the weights through LDS and split no outputs over
// workgroups ran these layers before; its waves sat idle 60-80% of the time.
// Measured against it (us, before -> after, MI355X, inputs from HBM): T = 16, 64 ->
// 64, 32,768 rows, fp32 134 -> 112 (bound now by the FP32 matrix rate, 53, and the
// staging beside it); T = 4, 192 -> 768, 25,216 rows, fp16 117 -> 72 (the L1
// path of the weight stream, 64 bytes a clock, and HBM, 37); T = 8, 96 -> 384,
// 12,608 rows, fp16 32 -> 29.5 (HBM 19); T = 7, 37 -> 53, 5,003 rows, fp16 18 -> 7.7;
// T = 13, 64 -> 338, 129 rows, bf16 134 -> 7.  At T = 8 the weights of a step come in
// two groups of planes: 123 registers against 208 with one group, three waves
// to a SIMD against two.
#pragma once
#include "eql_common.h"
#include "eql_config.h"
#include "eql_gemm.h"
#include "eql_launch.h"

namespace eqk {

template <int T, int DT>
struct XsShape {
  using Bn = Bins<T>;
  static constexpr bool W16 = DT != kF32;
  static constexpr int EB = W16 ? 2 : 4;
  static constexpr int KF = W16 ? 32 : 16;  // contraction channels per step
  static constexpr int KWM = W16 ? 8 : 4;   // of them per lane
  static constexpr int NB = 4 * T * EB;     // raw bytes of a staging unit: 4 channels of one row
  // groups of planes whose weights are loaded together (two register sets
  // alternate): one up to T = 4, two above
  static constexpr int NG = T > 4 ? 2 : 1;
  static constexpr int KB0 = NG == 1 ? Bn::K : Bn::K / 2;  // complex bins of group 0
  static constexpr int GS(int g) { return g == 0 ? 0 : Bn::R + 2 * KB0; }
  static constexpr int GE(int g) { return (NG == 1 || g == 1) ? T : Bn::R + 2 * KB0; }
  static constexpr int GP = NG == 1 ? T : (GE(0) > T - GE(0) ? GE(0) : T - GE(0));  // planes of the larger group
};

// LDS slot (bytes within a fragment block) of lane (g, i) at step ks.
__device__ __forceinline__ int xs_slot(int g, int i, int ks) { return (g * 16 + (i ^ (g | ((ks & 3) << 2)))) * 16; }

// Minimum waves per SIMD asked of the register allocator, and words of raw
// activations a thread keeps in flight while staging: what the accumulators (4
// T RT), two weight sets (8 GP) and, in chunks, the staging beside them leave
// room for without spilling.  The pipelined form runs eight waves a CU.
constexpr int xs_waves(int T, bool w16, int RT, int form) {
  if (form == kXsPipe) return 2;
  const bool chunk = form == kXsChunk;
  if (T * RT > 8) return RT == 4 || (chunk && T > 8) ? 2 : 3;
  return chunk ? (RT == 4 ? 2 : 3) : 4;
}
constexpr int xs_raw_words(int T, bool w16, int RT, int form) {
  return form == kXsChunk || xs_waves(T, w16, RT, form) == 4 ? 32 : 64;
}

// ODD: 16-bit elements and Ci * T odd, so that odd rows start at half a word.
// GATHER (forward of the group convolution, T in {1, 2, 4}): `in` is the
// feature map f [N pixels, geo.Cin, T] and row n is the patch row of pixel n
// (k*k*Cin channels: window orbits, then the centre), read straight from f.
// row0: first row of this launch; nks: steps run; nksw: steps of the stored
// weights; w_tiles: their tiles.
template <int T, int DT, bool BWD, int RT, bool ODD, bool GATHER, int FORM>
__global__ __launch_bounds__(512, xs_waves(T, DT != kF32, RT, FORM)) void eql_xs_kernel(
    const void* __restrict__ in, const void* __restrict__ wsp, const void* __restrict__ bias, void* __restrict__ out,
    int64_t N, int64_t row0, int Ci, int Co, int nks, int nksw, int kc, int n_ot, int osplit, int w_tiles,
    GatherGeom geo) {
  using S = XsShape<T, DT>;
  using Bn = Bins<T>;
  using FR = Frag<16>;
  using E = typename Elem<DT>::T;
  constexpr bool CHUNK = FORM == kXsChunk, PIPE = FORM == kXsPipe;
  constexpr int EB = S::EB;
  constexpr int NBW = S::NB / 4;
  constexpr int R = 16 * RT;
  static_assert(!ODD || (DT != kF32 && T % 2 == 1), "half-word rows");
  static_assert(!GATHER || (!BWD && !ODD && (T == 1 || T == 2 || T == 4)), "implicit gather");
  // [row tile][step][plane] blocks, then T times the bias of this workgroup's channels
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NW = nthr >> 6;
  const int g = lane >> 4;
  const int li = lane & 15;
  // the output splits of one row group run on one XCD (blocks are dealt
  // round-robin over the 8), so its rows come from that XCD's L2
  int os, rgp;
  {
    const int b = blockIdx.x, j = b >> 3;
    os = j % osplit;
    rgp = (j / osplit) * 8 + (b & 7);
  }
  if constexpr (PIPE) { os = 0; rgp = blockIdx.x; }
  int64_t r0 = row0 + (int64_t)rgp * R;
  if (r0 >= N) return;
  int len = N - r0 < R ? (int)(N - r0) : R;
  const int ot_lo = (int)((int64_t)os * n_ot / osplit), ot_hi = (int)((int64_t)(os + 1) * n_ot / osplit);
  const int rowb = Ci * T * EB;
  // The workgroup's rows as buffer resources: loads past them read zero,
  // stores past them are dropped.  (With half-word rows the range ends on the
  // word that holds the last element.)  GATHER: the whole feature map.
  __amdgpu_buffer_rsrc_t xrs =
      GATHER ? make_rsrc(in, (uint32_t)(N * geo.Cin * T * EB))
             : make_rsrc(reinterpret_cast<const char*>(in) + r0 * rowb, (uint32_t)((len * rowb + 3) & ~3));
  const __amdgpu_buffer_rsrc_t wrs = make_rsrc(wsp, (uint32_t)((int64_t)w_tiles * nksw * T * 1024));
  __amdgpu_buffer_rsrc_t ors =
      make_rsrc(reinterpret_cast<char*>(out) + r0 * Co * T * EB, (uint32_t)(len * Co * T * EB));
  const int xbytes = RT * kc * T * 1024;  // one staged spectrum
  float* const bl = reinterpret_cast<float*>(smem + (PIPE ? 2 : 1) * xbytes);

  // weights of (tile, step), planes of group G, into register set SI
  FR W[2][S::GP];
  auto load_w = [&](auto set, auto grp, int ot, int ks) __attribute__((always_inline)) {
    constexpr int G = decltype(grp)::value, SI = decltype(set)::value;
    const int soff = ((ot * nksw + ks) * T + S::GS(G)) * 1024;
    static_for<S::GE(G) - S::GS(G)>([&](auto pi) {
      constexpr int p = decltype(pi)::value;
      const u32x4 x = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16 + (p & 3) * 1024, soff + (p >> 2) * 4096, 0));
      W[SI][p].w[0] = x[0]; W[SI][p].w[1] = x[1]; W[SI][p].w[2] = x[2]; W[SI][p].w[3] = x[3];
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  int ot = ot_lo + wave;
  if (ot < ot_hi) load_w(I0{}, I0{}, ot, 0);

  // ---- staging.  A unit is 4 channels of one row; put() transforms the raw words
  // of unit (row, cq of the staged steps, which start at unit cq0 of a row) into base
  constexpr int RW = ODD ? NBW + 1 : NBW;
  auto put = [&](const uint32_t (&raw)[RW], int row, int cq, int cq0, bool plain, char* base) __attribute__((always_inline)) {
    uint32_t r[NBW];
    if constexpr (ODD) {
      const uint32_t sh = (row & 1) ? 16 : 0;
#pragma unroll
      for (int q = 0; q < NBW; ++q) r[q] = __builtin_amdgcn_alignbit(raw[q + 1], raw[q], sh);
    } else {
#pragma unroll
      for (int q = 0; q < NBW; ++q) r[q] = raw[q];
    }
    if constexpr (GATHER) gather_shear<T, 4, EB>(r, plain);
    if (Ci & 3) mask_raw<S::NB, EB>((Ci - 4 * (cq0 + cq)) * T, r);
    int ks, gg, hb;
    if constexpr (S::W16) { ks = cq >> 3; gg = (cq >> 1) & 3; hb = (cq & 1) * 8; }
    else { ks = cq >> 2; gg = cq & 3; hb = 0; }
    char* dst = base + (((row >> 4) * kc + ks) * T) * 1024 + xs_slot(gg, row & 15, ks) + hb;
    if constexpr (S::W16) {
      uint32_t P[T][2];
      if constexpr (DT == kF16) {
        raw_to_packed_planes<T, 4>(r, P);
      } else {
        float Q[T][4];
        raw_to_planes<T, DT, 4>(r, Q);
#pragma unroll
        for (int p = 0; p < T; ++p) { P[p][0] = pack2<DT>(Q[p][0], Q[p][1]); P[p][1] = pack2<DT>(Q[p][2], Q[p][3]); }
      }
#pragma unroll
      for (int p = 0; p < T; ++p) *reinterpret_cast<u32x2*>(dst + p * 1024) = u32x2{P[p][0], P[p][1]};
    } else {
      float Q[T][4];
      raw_to_planes<T, DT, 4>(r, Q);
#pragma unroll
      for (int p = 0; p < T; ++p)
        *reinterpret_cast<u32x4*>(dst + p * 1024) =
            u32x4{__builtin_bit_cast(uint32_t, Q[p][0]), __builtin_bit_cast(uint32_t, Q[p][1]),
                  __builtin_bit_cast(uint32_t, Q[p][2]), __builtin_bit_cast(uint32_t, Q[p][3])};
    }
  };
  // steps [k0, k0 + n), UB units in flight a thread
  auto stage = [&](int k0, int n) __attribute__((always_inline)) {
    constexpr int RAW = xs_raw_words(T, S::W16, RT, FORM);
    constexpr int UB = RW > RAW / 2 ? 1 : RW > RAW / 4 ? 2 : RW > RAW / 8 ? 4 : 8;
    const int CQ = n * (S::KF / 4), cq0 = k0 * (S::KF / 4);
    const int units = R * CQ;
    for (int u0 = tid; u0 < units; u0 += UB * nthr) {
      uint32_t raw[UB][RW];
      int row[UB], cq[UB];
      bool plain[UB];  // GATHER: the words are already in plain order (window centre)
#pragma unroll
      for (int v = 0; v < UB; ++v) {
        const int u = u0 + v * nthr;
        row[v] = (int)((unsigned)u / (unsigned)CQ);
        cq[v] = u - row[v] * CQ;
        plain[v] = true;
        if constexpr (GATHER) {
          const int c = 4 * (cq0 + cq[v]);
          gather_unit<T, EB>(xrs, geo, (uint32_t)(r0 + row[v]), (uint32_t)c, u < units && row[v] < len && c < Ci, raw[v],
                             plain[v]);
        } else {
          const bool ok = u < units && 4 * (cq0 + cq[v]) < Ci;
          const uint32_t off = ok ? (uint32_t)(row[v] * rowb + (cq0 + cq[v]) * S::NB) : kDropOffset;
          load_words<RW>(xrs, ODD ? off & ~3u : off, raw[v]);
        }
      }
#pragma unroll
      for (int v = 0; v < UB; ++v) {
        if (u0 + v * nthr >= units) break;
        put(raw[v], row[v], cq[v], cq0, plain[v], smem);
      }
    }
  };
  if constexpr (!BWD) {
    // a constant added to every group position is T times it added to bin 0
    const E* bp = reinterpret_cast<const E*>(bias);
    for (int i = tid; i < (ot_hi - ot_lo) * 16; i += nthr) {
      const int o = ot_lo * 16 + i;
      bl[i] = bp != nullptr && o < Co ? (float)T * (float)bp[o] : 0.0f;
    }
  }

  // ---- products.  The sign of each complex product sits on a negated operand:
  //   forward:  Re += Xr Wr + (-Xi) Wi,   Im += Xr Wi + Xi Wr
  //   backward: Re += Dr Wr + Di Wi,      Im += Di Wr + (-Dr) Wi
  floatx4 acc[T][RT];
  auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < T; ++p)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[p][r] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  const int xl = (g * 16 + (li ^ g)) * 16;
  const int rts = kc * T * 1024;
  int kb0 = 0;    // first step staged in LDS
  int xbuf = 0;   // PIPE: the buffer of the current chunk
  auto mma = [&](auto set, auto grp, int ksg) __attribute__((always_inline)) {
    constexpr int G = decltype(grp)::value, SI = decltype(set)::value;
    constexpr int gs = S::GS(G);
    const int ks = FORM != kXsWhole ? ksg - kb0 : ksg;
    const char* xb = smem + xbuf + (xl ^ ((ks & 3) << 6)) + ks * (T * 1024);  // xs_slot(g, li, ks)
    auto X = [&](int r, int p) __attribute__((always_inline)) {
      const u32x4 a = *reinterpret_cast<const u32x4*>(xb + r * rts + p * 1024);
      FR f;
      f.w[0] = a[0]; f.w[1] = a[1]; f.w[2] = a[2]; f.w[3] = a[3];
      return f;
    };
    // phase 0 of group 0: the real bins; then one phase per complex bin.  The
    // operands of the next phase are read ahead of the current one's products.
    constexpr int kb = G == 0 ? 0 : S::KB0, ke = G == 0 ? S::KB0 : Bn::K;
    constexpr int NPH = (ke - kb) + (G == 0 ? 1 : 0);
    FR xa[2][RT], xc[2][RT];
    auto read = [&](auto phi) __attribute__((always_inline)) {
      constexpr int ph = decltype(phi)::value;
      constexpr int Z = ph & 1;
      constexpr bool real = G == 0 && ph == 0;
      constexpr int k = kb + ph + (G == 0 ? 0 : 1);
      constexpr int p0 = real ? 0 : Bn::re(k), p1 = real ? 1 : Bn::im(k);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        xa[Z][r] = X(r, p0);
        if constexpr (!real || Bn::R == 2) xc[Z][r] = X(r, p1);
      }
    };
    read(I0{});
    static_for<NPH>([&](auto phi) {
      constexpr int ph = decltype(phi)::value;
      constexpr int Z = ph & 1;
      if constexpr (ph + 1 < NPH) read(std::integral_constant<int, ph + 1>{});
      if constexpr (G == 0 && ph == 0) {
#pragma unroll
        for (int r = 0; r < RT; ++r) frag_mma<DT, S::KWM>(acc[0][r], xa[Z][r], W[SI][0]);
        if constexpr (Bn::R == 2) {
#pragma unroll
          for (int r = 0; r < RT; ++r) frag_mma<DT, S::KWM>(acc[1][r], xc[Z][r], W[SI][1]);
        }
      } else {
        constexpr int k = kb + ph + (G == 0 ? 0 : 1);
        constexpr int re = Bn::re(k), im = Bn::im(k);
        const FR& wr = W[SI][re - gs];
        const FR& wi = W[SI][im - gs];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          frag_mma<DT, S::KWM>(acc[re][r], xa[Z][r], wr);
          if constexpr (!BWD) frag_mma<DT, S::KWM>(acc[im][r], xa[Z][r], wi);
          else frag_mma<DT, S::KWM>(acc[im][r], xc[Z][r], wr);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          if constexpr (!BWD) {
            frag_mma<DT, S::KWM>(acc[re][r], frag_neg<DT, 16>(xc[Z][r]), wi);
            frag_mma<DT, S::KWM>(acc[im][r], xc[Z][r], wr);
          } else {
            frag_mma<DT, S::KWM>(acc[re][r], xc[Z][r], wi);
            frag_mma<DT, S::KWM>(acc[im][r], frag_neg<DT, 16>(xa[Z][r]), wi);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // D = X W^T: lane (g, li) holds output channel 16 * tile + li of rows 4g .. 4g+3
  // of each row tile; the 16 lanes of a lane group store 16 consecutive
  // channels of one row (16 * T contiguous elements)
  auto epilogue = [&](int t) __attribute__((always_inline)) {
    const int o = t * 16 + li;
    float bv = 0.0f;
    if constexpr (!BWD) bv = bl[o - ot_lo * 16];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rt * 16 + 4 * g + r;
        float Pl[T], ul[T];
#pragma unroll
        for (int p = 0; p < T; ++p) Pl[p] = acc[p][rt][r];
        if constexpr (!BWD) Pl[0] += bv;
        irdft<T>(Pl, ul);
        const uint32_t off = (row < len && o < Co) ? (uint32_t)((row * Co + o) * T * EB) : kDropOffset;
        store_run_rsrc<DT, T>(ors, off, ul);
      }
  };
  int ks = 0;
  auto step = [&](auto par) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
    int k1 = ks + 1, o1 = ot;
    if (k1 == nks) { k1 = 0; if constexpr (!PIPE) o1 += NW; }
    const int ol = o1 < ot_hi ? o1 : ot;  // past the last tile: a valid block, never used
    if constexpr (S::NG == 1) {
      load_w(std::integral_constant<int, 1 - P>{}, I0{}, ol, k1);
      __builtin_amdgcn_sched_barrier(0);
      mma(std::integral_constant<int, P>{}, I0{}, ks);
    } else {
      load_w(I1{}, I1{}, ot, ks);
      __builtin_amdgcn_sched_barrier(0);
      mma(I0{}, I0{}, ks);
      load_w(I0{}, I0{}, ol, k1);
      __builtin_amdgcn_sched_barrier(0);
      mma(I1{}, I1{}, ks);
    }
    if (k1 == 0) {
      epilogue(ot);
      zero_acc();
    }
    ks = k1;
    ot = o1;
  };
  // `left` steps from (ot, ks), the two weight sets in turn
  auto run = [&](int left) __attribute__((always_inline)) {
    while (left > 0) {
      step(I0{});
      if (--left == 0) break;
      if constexpr (S::NG == 1) {
        step(I1{});
        --left;
      }
    }
  };
  if constexpr (FORM == kXsWhole) {
    // all steps staged at once: a wave runs every NW-th output tile of the workgroup
    stage(0, nks);
    __syncthreads();
    zero_acc();
    if (ot < ot_hi) run((ot_hi - ot + NW - 1) / NW * nks);
  } else if constexpr (CHUNK) {
    // chunks of kc steps (kc even, so each starts at weight set 0) staged in
    // turn; a wave keeps its one tile's accumulators across them (the host
    // gives a workgroup at most NW tiles)
    zero_acc();
    for (int k0 = 0; k0 < nks; k0 += kc) {
      const int n = nks - k0 < kc ? nks - k0 : kc;
      if (k0 > 0) __syncthreads();  // the previous chunk read everywhere
      stage(k0, n);
      __syncthreads();
      kb0 = k0;
      if (ot < ot_hi) run(n);
    }
  } else {
    // A workgroup walks its row groups (every gridDim'th) and their chunks.  Wave w <
    // n_ot runs the products of output tile w, the others stage: in turn `it`
    // they write chunk `it` into one LDS buffer while the products of chunk it - 1
    // read the other.  Both sides count the same turns, one barrier each; no
    // wait at a barrier for loads in flight, which are the wave's own.
    static_assert(!GATHER && !ODD && S::NG == 2, "pipelined form");
    constexpr int UB = xs_pipe_units(T);
    const int nch = (nks + kc - 1) / kc;
    const int64_t groups = (N + R - 1) / R;
    const int64_t turns = (groups - 1 - blockIdx.x) / gridDim.x + 1;
    const int64_t total = turns * nch;
    auto rows = [&](int64_t grp) __attribute__((always_inline)) {
      r0 = grp * R;
      len = N - r0 < R ? (int)(N - r0) : R;
    };
    auto turn = [&]() __attribute__((always_inline)) {
      __builtin_amdgcn_s_waitcnt(0xc07f);  // LDS reads and writes done; loads and stores stay in flight
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      __builtin_amdgcn_s_barrier();
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
    };
    int64_t grp = blockIdx.x;
    int k0 = 0;
    if (wave < n_ot) {
      zero_acc();
      for (int64_t it = 0; it <= total; ++it) {
        if (it > 0) {
          xbuf = (it & 1) ? 0 : xbytes;
          kb0 = k0;
          run(nks - k0 < kc ? nks - k0 : kc);
          k0 += kc;
          if (k0 >= nks) {
            k0 = 0;
            grp += gridDim.x;
            if (grp < groups) {
              rows(grp);
              ors = make_rsrc(reinterpret_cast<char*>(out) + r0 * Co * T * EB, (uint32_t)(len * Co * T * EB));
            }
          }
        }
        turn();
      }
    } else {
      const int pt = tid - n_ot * 64, npt = nthr - n_ot * 64;
      const int CQ = kc * (S::KF / 4), units = R * CQ;
      uint32_t raw[UB][RW];
      int row[UB], cq[UB];
#pragma unroll
      for (int v = 0; v < UB; ++v) {
        const int u = pt + v * npt;
        row[v] = (int)((unsigned)u / (unsigned)CQ);
        cq[v] = u - row[v] * CQ;
      }
      auto load = [&](int v) __attribute__((always_inline)) {
        const int c = k0 * (S::KF / 4) + cq[v];
        const bool ok = row[v] < R && 4 * c < Ci && grp < groups;
        load_words<RW>(xrs, ok ? (uint32_t)(row[v] * rowb + c * S::NB) : kDropOffset, raw[v]);
      };
#pragma unroll
      for (int v = 0; v < UB; ++v) load(v);
      for (int64_t it = 0; it <= total; ++it) {
        if (it < total) {
          const int cq0 = k0 * (S::KF / 4);
          k0 += kc;
          if (k0 >= nks) {
            k0 = 0;
            grp += gridDim.x;
            if (grp < groups) {
              rows(grp);
              xrs = make_rsrc(reinterpret_cast<const char*>(in) + r0 * rowb, (uint32_t)(len * rowb));
            }
          }
#pragma unroll
          for (int v = 0; v < UB; ++v) {
            if (pt + v * npt < units) put(raw[v], row[v], cq[v], cq0, true, smem + ((it & 1) ? xbytes : 0));
            load(v);  // the next chunk's rows
          }
        }
        turn();
      }
    }
  }
}

}  // namespace eqk

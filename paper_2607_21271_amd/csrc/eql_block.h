// eql_block.h -- the encoder block around the equivariant layers, for gfx950:
// layer norm over (channel, group) rows and softmax attention over one
// image's tokens, each in one pass over memory (inference of the drop-in block
// of Sec. 4.2).
#pragma once
#include "eql_common.h"
#include "eql_config.h"
#include "eql_gemm.h"
#include "eql_launch.h"

namespace eqk {

// ---- layer norm ------------------------------------------------------------
// y = (x - mean) / sqrt(var + eps) * weight[c] + bias[c] over the C * T
// contiguous elements of a row, mean and then squared deviations in fp32 from
// the row held in registers, one rounding at the end.  WPR waves hold a row, V
// 16-byte vectors a lane (lane l: vectors l, l + 64 WPR, ...); a wave keeps
// its weight and bias in registers and takes every gridDim'th row.
// 25,216 rows of 768 fp16 elements 26 us, 3.0 TB/s, against 4.9 TB/s of a pass
// that streams equal bytes in and out: a wave has no load in flight during
// its row's two reductions.  torch's eleven operations took about 230 us.
template <int DT, int V, int WPR>
__global__ __launch_bounds__(256) void eql_group_norm_kernel(const void* __restrict__ x, const void* __restrict__ weight,
                                                             const void* __restrict__ bias, void* __restrict__ y,
                                                             int64_t rows, int T, int C, float eps) {
  using E = typename Elem<DT>::T;
  constexpr int VEC = DT == kF32 ? 4 : 8;
  constexpr int RPB = 4 / WPR;  // rows of a workgroup
  __shared__ float red[2][4];
  const int n = C * T, nv = n / VEC;
  const int wave = threadIdx.x >> 6;
  const int l = threadIdx.x & (64 * WPR - 1);
  float wv[V][VEC], bv[V][VEC];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int e0 = (v * 64 * WPR + l) * VEC;
    int c = (int)((unsigned)e0 / (unsigned)T), t = e0 - c * T;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      const bool ok = c < C;
      wv[v][i] = ok ? (float)reinterpret_cast<const E*>(weight)[c] : 0.0f;
      bv[v][i] = ok ? (float)reinterpret_cast<const E*>(bias)[c] : 0.0f;
      if (++t == T) { t = 0; ++c; }
    }
  }
  auto total = [&](float s, int slot) {
#pragma unroll
    for (int d = 1; d < 64; d *= 2) s += __shfl_xor(s, d);
    if constexpr (WPR > 1) {
      if ((threadIdx.x & 63) == 0) red[slot][wave] = s;
      __syncthreads();
      s = (red[slot][0] + red[slot][1]) + (red[slot][2] + red[slot][3]);
    }
    return s;
  };
  for (int64_t r = (int64_t)blockIdx.x * RPB + (WPR == 1 ? wave : 0); r < rows; r += (int64_t)gridDim.x * RPB) {
    const u32x4* src = reinterpret_cast<const u32x4*>(reinterpret_cast<const E*>(x) + r * n);
    u32x4* dst = reinterpret_cast<u32x4*>(reinterpret_cast<E*>(y) + r * n);
    u32x4 in[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int i = v * 64 * WPR + l;
      in[v] = i < nv ? src[i] : u32x4{0, 0, 0, 0};
    }
    float f[V][VEC], s = 0.0f;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const uint32_t w[4] = {in[v][0], in[v][1], in[v][2], in[v][3]};
      raw_to_floats<DT, 4>(w, f[v]);
#pragma unroll
      for (int i = 0; i < VEC; ++i) s += f[v][i];
    }
    const float mu = total(s, 0) / (float)n;
    s = 0.0f;
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        f[v][i] -= mu;
        if (v * 64 * WPR + l < nv) s += f[v][i] * f[v][i];
      }
    const float rs = 1.0f / sqrtf(total(s, 1) / (float)n + eps);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int i = v * 64 * WPR + l;
#pragma unroll
      for (int j = 0; j < VEC; ++j) f[v][j] = f[v][j] * rs * wv[v][j] + bv[v][j];
      u32x4 out;
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = pack2<DT>(f[v][j * VEC / 4], f[v][(j * VEC + VEC / 2) / 4]);
      if (i < nv) dst[i] = out;
    }
  }
}

// ---- attention -------------------------------------------------------------
// o[b, q, h, :] = sum_k softmax_k(scale q . k) v over the L <= 32 KT tokens of
// one image, qkv [B, L, 3, H, D] as the qkv layer writes it, o [B, L, H, D];
// 16-bit elements, D in {32, 64, 128}.
//
// A workgroup of four or eight waves stages K (rows) and V (transposed) of one (image,
// head) in LDS and its waves take tiles of 16 queries.  The scores are computed
// transposed, S^T = K Q^T, so that a lane holds keys 16 t + 4 g + r of the one
// query li: the row maximum and sum are two shuffles, and two score tiles are
// directly the B operand of O^T = V^T P^T once V^T's columns are stored in the
// same order (vt_slot).  No score leaves the registers; scores, softmax and sums
// are fp32, the probabilities are rounded once to the element type.
//
// It replaces three copies, two batched products and a scaled fp32 softmax
// between them, which moved the score matrix through memory nine times.  Bound
// by the exponentials and the staging; 128 images of 197 tokens, 12 heads of
// 64, fp16: 49 us for 155 MB (3.2 TB/s) against about 680 us.  The norm and
// this kernel together take the whole encoder block from 1576 to 430 us.
constexpr int attn_k_pitch(int D) { return D * 2 + 16; }
constexpr int attn_v_pitch(int KT) { return KT * 64 + 16; }
constexpr int attn_lds_bytes(int D, int KT) { return KT * 32 * attn_k_pitch(D) + D * attn_v_pitch(KT); }

// waves of a workgroup: at the long sequences one or two workgroups fit a CU's LDS
constexpr int attn_waves(int KT) { return KT > 4 ? 8 : 4; }

template <int DT, int D, int KT>
__global__ __launch_bounds__(attn_waves(KT) * 64, 2) void eql_attention_kernel(const void* __restrict__ qkv, void* __restrict__ o, int L,
                                                               int H, float scale_log2e, int qsplit) {
  using FR = Frag<16>;
  constexpr int DS = D / 32;  // contraction steps of a score
  constexpr int DC = D / 8;   // 16-byte chunks of a row
  constexpr int KP = attn_k_pitch(D), VP = attn_v_pitch(KT);
  constexpr int NW = attn_waves(KT), NT = NW * 64;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* const ks = smem;
  char* const vs = smem + KT * 32 * KP;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, li = lane & 15;
  const int bh = blockIdx.x / qsplit, part = blockIdx.x % qsplit;
  const int b = bh / H, h = bh % H;
  const int64_t rs = (int64_t)3 * H * D;
  const uint16_t* const q = reinterpret_cast<const uint16_t*>(qkv) + (int64_t)b * L * rs + h * D;
  const uint16_t* const k = q + H * D;
  const uint16_t* const v = k + H * D;
  auto chunk = [&](const uint16_t* p, int row, int c) {  // rows past L read row L - 1
    return *reinterpret_cast<const u32x4*>(p + (int64_t)(row < L ? row : L - 1) * rs + c * 8);
  };
  constexpr int KUr = (KT * 32 * DC + NT - 1) / NT;
  constexpr int VUr = (KT * 16 * DC + NT - 1) / NT;
  {
    u32x4 kr[KUr], va[VUr], vb[VUr];
#pragma unroll
    for (int i = 0; i < KUr; ++i) {
      const int u = tid + i * NT;
      kr[i] = chunk(k, u / DC, u % DC);
    }
    if constexpr (KT * D > NT) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < VUr; ++i) {
      const int u = tid + i * NT;
      va[i] = chunk(v, 2 * (u / DC), u % DC);
      vb[i] = chunk(v, 2 * (u / DC) + 1, u % DC);
    }
#pragma unroll
    for (int i = 0; i < KUr; ++i) {
      const int u = tid + i * NT, key = u / DC;
      if (key < KT * 32)
        *reinterpret_cast<u32x4*>(ks + key * KP + (u % DC) * 16) = key < L ? kr[i] : u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int i = 0; i < VUr; ++i) {
      const int u = tid + i * NT, key = 2 * (u / DC);
      if (key >= KT * 32) continue;
      // vt_slot: key 32 s + 16 a + 4 g + r at column 32 s + 8 g + 4 a + r
      const int slot = (key & ~31) + ((key >> 2) & 3) * 8 + ((key >> 4) & 1) * 4 + (key & 3);
      char* dst = vs + (u % DC) * 8 * VP + slot * 2;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint32_t x0 = key < L ? va[i][m] : 0u, x1 = key + 1 < L ? vb[i][m] : 0u;
        *reinterpret_cast<uint32_t*>(dst + (2 * m) * VP) = (x0 & 0xffffu) | (x1 << 16);
        *reinterpret_cast<uint32_t*>(dst + (2 * m + 1) * VP) = (x0 >> 16) | (x1 & 0xffff0000u);
      }
    }
  }
  __syncthreads();
  auto frag = [&](const void* p) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(p);
    FR f;
    f.w[0] = a[0]; f.w[1] = a[1]; f.w[2] = a[2]; f.w[3] = a[3];
    return f;
  };
  const int nq = (L + 15) / 16;
  for (int qt = part * NW + wave; qt < nq; qt += NW * qsplit) {
    const int row = qt * 16 + li;
    asm volatile("" ::: "memory");  // K and V^T are read from LDS for each tile, not kept in registers
    FR qf[DS];
#pragma unroll
    for (int s = 0; s < DS; ++s) qf[s] = frag(q + (int64_t)(row < L ? row : L - 1) * rs + s * 32 + g * 8);
    floatx4 sc[2 * KT];
    float mx = -__builtin_inff();
#pragma unroll
    for (int t = 0; t < 2 * KT; ++t) {
      sc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < DS; ++s) frag_mma<DT, 8>(sc[t], frag(ks + (t * 16 + li) * KP + s * 64 + g * 16), qf[s]);
      if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the fragments in flight
    }
#pragma unroll
    for (int t = 0; t < 2 * KT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // L > 32 (KT - 1): only the last two tiles hold keys past it
        if (t >= 2 * KT - 2 && t * 16 + 4 * g + r >= L) sc[t][r] = -__builtin_inff();
        mx = fmaxf(mx, sc[t][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < 2 * KT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[t][r] = __builtin_amdgcn_exp2f((sc[t][r] - mx) * scale_log2e);
        sum += sc[t][r];
      }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    const float inv = 1.0f / sum;
    FR pf[KT];
#pragma unroll
    for (int s = 0; s < KT; ++s)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const floatx4& p = sc[2 * s + w / 2];
        pf[s].w[w] = pack2<DT>(p[2 * (w & 1)] * inv, p[2 * (w & 1) + 1] * inv);
      }
    uint16_t* const dst = reinterpret_cast<uint16_t*>(o) + (((int64_t)b * L + row) * H + h) * D + 4 * g;
#pragma unroll
    for (int d = 0; d < D / 16; ++d) {
      floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KT; ++s) frag_mma<DT, 8>(acc, frag(vs + (d * 16 + li) * VP + s * 64 + g * 16), pf[s]);
      if (d % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      if (row < L)
        *reinterpret_cast<u32x2*>(dst + d * 16) = u32x2{pack2<DT>(acc[0], acc[1]), pack2<DT>(acc[2], acc[3])};
    }
  }
}

}  // namespace eqk

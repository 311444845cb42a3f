// eql_block.hip -- instantiations and launches of the encoder block's kernels
// (eql_block.h).
#include "eql_block.h"

namespace eqk {
namespace {

template <int DT, int WPR>
hipError_t norm_v(const void* x, const void* w, const void* b, void* y, int64_t rows, int T, int C, float eps, int cus,
                  hipStream_t stream) {
  const int nv = C * T / (DT == kF32 ? 4 : 8);
  const int V = (nv + 64 * WPR - 1) / (64 * WPR);
  const int rpb = 4 / WPR;
  int64_t grid = (rows + rpb - 1) / rpb;
  if (grid > (int64_t)cus * 8) grid = (int64_t)cus * 8;  // resident workgroups: weights read once by each
#define EQL_NORM(v)                                                                                             \
  hipLaunchKernelGGL((eql_group_norm_kernel<DT, v, WPR>), dim3((unsigned)grid), dim3(256), 0, stream, x, w, b, y, \
                     rows, T, C, eps)
  switch (V) {
    case 1: EQL_NORM(1); break;
    case 2: EQL_NORM(2); break;
    case 3: EQL_NORM(3); break;
    case 4: EQL_NORM(4); break;
    default: return hipErrorInvalidValue;
  }
#undef EQL_NORM
  return hipGetLastError();
}

// One wave holds a row of up to 4 vectors a lane; four waves one of up to four times that.
template <int DT>
hipError_t norm_dt(const void* x, const void* w, const void* b, void* y, int64_t rows, int T, int C, float eps, int cus,
                   hipStream_t stream) {
  if (C * T <= kNormMaxBytes / 4 / (DT == kF32 ? 4 : 2))
    return norm_v<DT, 1>(x, w, b, y, rows, T, C, eps, cus, stream);
  return norm_v<DT, 4>(x, w, b, y, rows, T, C, eps, cus, stream);
}

template <int DT, int D, int KT>
hipError_t attn_kt(const void* qkv, void* o, int64_t B, int L, int H, float scale, int cus, hipStream_t stream) {
  if constexpr (KT > kAttnMaxL / 32) {
    return hipErrorInvalidValue;
  } else {
    if (L > 32 * KT) return attn_kt<DT, D, KT + 1>(qkv, o, B, L, H, scale, cus, stream);
    auto k = eql_attention_kernel<DT, D, KT>;
    constexpr int lds = attn_lds_bytes(D, KT);
    if constexpr (lds > 65536) {
      const hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
    }
    // With fewer (image, head) pairs than workgroups fit the device, the query tiles
    // of one are split, each part staging K and V again.  Two workgroups fit a
    // CU, one where K and V^T take more than half its LDS (head_dim 128 past 128
    // tokens: 390 pairs of 150 tokens, fp16, in two parts 37 us, in one 28).
    constexpr int resident = 2 * lds <= kLdsBytes ? 2 : 1;
    int64_t qs = (resident * (int64_t)cus + B * H - 1) / (B * H);
    const int max_qs = ((L + 15) / 16 + attn_waves(KT) - 1) / attn_waves(KT);
    if (qs > max_qs) qs = max_qs;
    const int64_t most = launch_blocks(attn_waves(KT) * 64) / (H * qs);  // images of one launch
    for (int64_t b0 = 0; b0 < B; b0 += most) {
      const int64_t n = B - b0 < most ? B - b0 : most;
      hipLaunchKernelGGL(k, dim3((unsigned)(n * H * qs)), dim3(attn_waves(KT) * 64), lds, stream,
                         (const char*)qkv + b0 * L * 6 * H * D, (char*)o + b0 * L * 2 * H * D, L, H,
                         scale * 1.4426950408889634f, (int)qs);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
}

template <int DT>
hipError_t attn_dt(const void* qkv, void* o, int64_t B, int L, int H, int D, float scale, int cus, hipStream_t stream) {
  if (D == 32) return attn_kt<DT, 32, 1>(qkv, o, B, L, H, scale, cus, stream);
  if (D == 64) return attn_kt<DT, 64, 1>(qkv, o, B, L, H, scale, cus, stream);
  if (D == 128) return attn_kt<DT, 128, 1>(qkv, o, B, L, H, scale, cus, stream);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_group_norm(int dt, const void* x, const void* w, const void* b, void* y, int64_t rows, int T, int C,
                             float eps, int cus, hipStream_t stream) {
  if (dt == kF32) return norm_dt<kF32>(x, w, b, y, rows, T, C, eps, cus, stream);
  if (dt == kF16) return norm_dt<kF16>(x, w, b, y, rows, T, C, eps, cus, stream);
  return norm_dt<kBF16>(x, w, b, y, rows, T, C, eps, cus, stream);
}

hipError_t launch_attention(int dt, const void* qkv, void* o, int64_t B, int L, int H, int D, float scale, int cus,
                            hipStream_t stream) {
  return dt == kF16 ? attn_dt<kF16>(qkv, o, B, L, H, D, scale, cus, stream)
                    : attn_dt<kBF16>(qkv, o, B, L, H, D, scale, cus, stream);
}

}  // namespace eqk

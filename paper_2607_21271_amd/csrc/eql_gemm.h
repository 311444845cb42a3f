// eql_gemm.h -- device helpers shared by the MFMA kernels of the C_T
// equivariant linear layer for gfx950: operand fragments and their products,
// swizzled LDS rows, buffer loads and stores, raw words to spectral planes, and
// the implicit patch gather of the group convolution.
#pragma once
#include "eql_common.h"
#include "eql_config.h"

namespace eqk {

template <int FB>
struct Frag {
  uint32_t w[FB / 4];
};

template <int DT, int KW>
__device__ __forceinline__ void frag_mma(floatx4& acc, const Frag<KW*(DT != kF32 ? 2 : 4)>& a,
                                         const Frag<KW*(DT != kF32 ? 2 : 4)>& b) {
  if constexpr (DT == kF16 && KW == 8) {
    const u32x4 av = {a.w[0], a.w[1], a.w[2], a.w[3]};
    const u32x4 bv = {b.w[0], b.w[1], b.w[2], b.w[3]};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, av),
                                                 __builtin_bit_cast(half8, bv), acc, 0, 0, 0);
  } else if constexpr (DT == kBF16 && KW == 8) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    const u32x4 av = {a.w[0], a.w[1], a.w[2], a.w[3]};
    const u32x4 bv = {b.w[0], b.w[1], b.w[2], b.w[3]};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                  __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
  } else {
    static_assert(DT == kF32, "16-bit fragments hold eight channels a lane");
#pragma unroll
    for (int s = 0; s < KW; ++s)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.w[s]),
                                                 __builtin_bit_cast(float, b.w[s]), acc, 0, 0, 0);
  }
}

// sign flip of every element (the sign is the top bit of fp16, bf16 and fp32)
template <int DT, int FB>
__device__ __forceinline__ Frag<FB> frag_neg(const Frag<FB>& a) {
  Frag<FB> r;
#pragma unroll
  for (int j = 0; j < FB / 4; ++j) r.w[j] = a.w[j] ^ (DT != kF32 ? 0x80008000u : 0x80000000u);
  return r;
}

// Swizzled LDS rows of RB bytes: 16-byte chunk c of row r lives at chunk
// c ^ ((r >> 1) & (RB/16 - 1)).
template <int RB>
__device__ __forceinline__ int wl_off(int row, int byte) {
  constexpr int NCH = RB / 16;
  const int ch = byte >> 4;
  return row * RB + ((ch ^ ((row >> 1) & (NCH - 1))) << 4) + (byte & 15);
}

template <int FB, int RB>
__device__ __forceinline__ Frag<FB> lds_frag(const char* base, int row, int g) {
  static_assert(FB == 16, "fragment size");
  Frag<FB> f;
  const u32x4 a = *reinterpret_cast<const u32x4*>(base + wl_off<RB>(row, g * 16));
  f.w[0] = a[0]; f.w[1] = a[1]; f.w[2] = a[2]; f.w[3] = a[3];
  return f;
}

// Buffer resource over [base, base + bytes): loads past the end return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// One lane's L contiguous output elements through a buffer resource, at byte
// offset off; a lane passes kDropOffset (past any resource) to store nothing.
// No branch skips a store, so every path through a loop issues the same
// memory operations and the compiler's memory-counter waits stay exact.
constexpr uint32_t kDropOffset = 0x80000000u;
template <int DT, int L>
__device__ __forceinline__ void store_run_rsrc(__amdgpu_buffer_rsrc_t rs, uint32_t off, const float (&v)[L]) {
  using E = typename Elem<DT>::T;
  constexpr int EBY = Elem<DT>::bytes;
  constexpr int NB = L * EBY;
  constexpr int VEC = (NB % 16 == 0) ? 16 : (NB % 8 == 0) ? 8 : (NB % 4 == 0) ? 4 : 2;
  constexpr int PER = VEC / EBY;
#pragma unroll
  for (int s = 0; s < L / PER; ++s) {
    E tmp[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) tmp[q] = (E)v[s * PER + q];
    const uint32_t o = off + s * VEC;
    if constexpr (VEC == 16) {
      u32x4 w;
      __builtin_memcpy(&w, tmp, 16);
      __builtin_amdgcn_raw_buffer_store_b128(w, rs, o, 0, 0);
    } else if constexpr (VEC == 8) {
      u32x2 w;
      __builtin_memcpy(&w, tmp, 8);
      __builtin_amdgcn_raw_buffer_store_b64(w, rs, o, 0, 0);
    } else if constexpr (VEC == 4) {
      uint32_t w;
      __builtin_memcpy(&w, tmp, 4);
      __builtin_amdgcn_raw_buffer_store_b32(w, rs, o, 0, 0);
    } else {
      uint16_t w;
      __builtin_memcpy(&w, tmp, 2);
      __builtin_amdgcn_raw_buffer_store_b16(w, rs, o, 0, 0);
    }
  }
}

// NW words from byte offset off (a multiple of 4) of the resource, in the widest
// loads: a buffer load of two to four words needs word alignment only, and each
// word past the resource reads as zero.  One load shape per kernel: with the
// width chosen at run time among several load shapes feeding the same
// registers, the register allocator in this toolchain produced code that
// overwrote live raw words in some kernels.
template <int NW>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t (&r)[NW]) {
  constexpr int Q = NW / 4;
#pragma unroll
  for (int v = 0; v < Q; ++v) {
    const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * v, 0, 0));
    r[4 * v] = x[0]; r[4 * v + 1] = x[1]; r[4 * v + 2] = x[2]; r[4 * v + 3] = x[3];
  }
  if constexpr (NW % 4 >= 2) {
    const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, off + 16 * Q, 0, 0));
    r[4 * Q] = x[0]; r[4 * Q + 1] = x[1];
  }
  if constexpr (NW % 2 == 1) r[NW - 1] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4 * (NW - 1), 0, 0);
}

// Zero the elements past nvalid (a ragged last channel group).
template <int NB, int EB>
__device__ __forceinline__ void mask_raw(int nvalid_elems, uint32_t (&r)[NB / 4]) {
  if (nvalid_elems >= NB / EB) return;
#pragma unroll
  for (int v = 0; v < NB / 4; ++v) {
    if constexpr (EB == 2) {
      if (2 * v + 1 >= nvalid_elems) r[v] = (2 * v < nvalid_elems) ? (r[v] & 0xffffu) : 0u;
    } else {
      if (v >= nvalid_elems) r[v] = 0u;
    }
  }
}

// Implicit patch gather (group convolution): a lane's raw words hold T
// vectors, vector j being the HKW elements vec_j[cc*T + s] = f[pixel + R^j d0,
// c + cc, s] of one window orbit (M = HKW / T input channels c + cc, every
// group position s).  The gathered channel (cc, u) at group position j is
// vec_j[cc*T + (u + j) mod T] (the shear u = s - j); this rewrites the words
// into the plain order, element (cc*T + u)*T + j.  The centre of the window is
// already in plain order (keep).
template <int T, int HKW, int EB>
__device__ __forceinline__ void gather_shear(uint32_t (&r)[HKW * T * EB / 4], bool keep) {
  constexpr int NW = HKW * T * EB / 4;
  // source element of plain element i = (cc*T + u)*T + j
  constexpr auto src = [](int i) {
    const int j = i % T, u = (i / T) % T, cc = i / (T * T);
    return j * HKW + cc * T + (u + j) % T;
  };
  // every index below is a compile-time constant: the sheared words are
  // built into their own array and the lane's choice applied per word (a
  // per-element choice of source index became a runtime-indexed array)
  uint32_t o[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if constexpr (EB == 4) {
      o[w] = r[src(w)];
    } else {
      const int s0 = src(2 * w), s1 = src(2 * w + 1);
      const uint32_t lo = (r[s0 / 2] >> (16 * (s0 % 2))) & 0xffffu;
      const uint32_t hi = (r[s1 / 2] >> (16 * (s1 % 2))) & 0xffffu;
      o[w] = lo | (hi << 16);
    }
  }
  const uint32_t km = keep ? 0xffffffffu : 0u;
#pragma unroll
  for (int w = 0; w < NW; ++w) r[w] = (r[w] & km) | (o[w] & ~km);
}

// n / d and n mod d for n < 2^31 and a launch-constant divisor d with its
// multiplier m = floor(2^32 / d) (2^32 - 1 for d = 1): the product estimate
// is exact or one low
__device__ __forceinline__ uint32_t gather_div(uint32_t n, uint32_t d, uint32_t m, uint32_t& r) {
  uint32_t q = __umulhi(n, m);
  r = n - q * d;
  if (r >= d) {
    ++q;
    r -= d;
  }
  return q;
}

// Raw words of one lane's gathered channels: HKW = 4 channels cabs.. of the
// patch row of pixel p, T loads of 4 elements each.  They are 4 / T input
// channels c.. of one window orbit O (all T sheared positions), or 4 channels
// of the centre (plain).  The host keeps Cin a multiple of 4, so a lane never
// straddles two blocks.  Pixels outside the image and lanes with ok false
// (rows past the workgroup's, channels past k*k*Cin) read zero (dropped
// offsets).  Divisions by launch constants are multiplies (GatherGeom),
// offsets 32-bit (the feature map is below 2^31 bytes).
template <int T, int EB>
__device__ __forceinline__ void gather_unit(__amdgpu_buffer_rsrc_t xrs, const GatherGeom& geo, uint32_t p,
                                            uint32_t cabs, bool row_ok, uint32_t (&r)[T * EB], bool& plain) {
  constexpr int VB = 4 * EB;  // bytes per vector
  const uint32_t CT = (uint32_t)geo.Cin * T;
  uint32_t x, y, rem;
  const uint32_t py = gather_div(p, (uint32_t)geo.W, geo.mW, x);
  gather_div(py, (uint32_t)geo.H, geo.mH, y);
  uint32_t cr;
  const uint32_t O = gather_div(cabs, CT, geo.mCT, cr);
  const int h = geo.k >> 1;
  const bool centre = (int)O >= (geo.k * geo.k - 1) / T;  // past the last orbit block
  // orbit base point (a0, b0)
  int a0, b0;
  if constexpr (T == 4) {
    const uint32_t qa = gather_div(O, (uint32_t)(h + 1), geo.mO, rem);
    a0 = 1 + (int)qa;
    b0 = (int)rem;
  } else if constexpr (T == 2) {
    const uint32_t qa = gather_div(O, (uint32_t)geo.k, geo.mO, rem);
    const bool upper = (int)qa < h;
    a0 = upper ? 1 + (int)qa : 0;
    b0 = upper ? (int)rem - h : 1 + (int)rem;
  } else {
    const uint32_t idx = O + (O >= (uint32_t)((geo.k * geo.k - 1) / 2) ? 1u : 0u);
    const uint32_t qa = gather_div(idx, (uint32_t)geo.k, geo.mO, rem);
    a0 = (int)qa - h;
    b0 = (int)rem - h;
  }
  if (centre) { a0 = 0; b0 = 0; }
  // byte offset of the lane's first channel in a pixel row: orbit lanes
  // read channel c = cr / T of T pixels, centre lanes T consecutive
  // vectors of their own pixel
  const uint32_t coff = centre ? (cabs - O * CT) * T * EB : (cr / T) * T * EB;
  const uint32_t rowf = CT * EB;
  plain = centre;
  static_for<T>([&](auto ji) {
    constexpr int j = decltype(ji)::value;
    // R^j (a0, b0): R(a, b) = (-b, a) at T = 4, (-a, -b) at T = 2
    int a = a0, b = b0;
    if constexpr (T == 4) {
      if constexpr (j == 1) { a = -b0; b = a0; }
      if constexpr (j == 2) { a = -a0; b = -b0; }
      if constexpr (j == 3) { a = b0; b = -a0; }
    } else if constexpr (T == 2) {
      if constexpr (j == 1) { a = -a0; b = -b0; }
    }
    const bool in_img = (uint32_t)((int)y + a) < (uint32_t)geo.H && (uint32_t)((int)x + b) < (uint32_t)geo.W;
    const uint32_t pix = p + (uint32_t)(a * geo.W + b);
    const uint32_t off = (row_ok && in_img) ? pix * rowf + coff + (centre ? (uint32_t)(j * VB) : 0u)
                                            : kDropOffset;
    if constexpr (VB == 16) {
      const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrs, off, 0, 0));
      r[4 * j] = v[0]; r[4 * j + 1] = v[1]; r[4 * j + 2] = v[2]; r[4 * j + 3] = v[3];
    } else {
      static_assert(VB == 8, "gather vector");
      const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(xrs, off, 0, 0));
      r[2 * j] = v[0]; r[2 * j + 1] = v[1];
    }
  });
}

// Transform the HKW channels held raw by one lane; P[p][j] is plane p of channel j.
template <int T, int DT, int HKW>
__device__ __forceinline__ void raw_to_planes(const uint32_t (&r)[HKW * T * (DT != kF32 ? 2 : 4) / 4],
                                              float (&P)[T][HKW]) {
  constexpr int NW = HKW * T * (DT != kF32 ? 2 : 4) / 4;
  float f[DT != kF32 ? 2 * NW : NW];
  raw_to_floats<DT, NW>(r, f);
#pragma unroll
  for (int j = 0; j < HKW; ++j) {
    float v[T], q[T];
#pragma unroll
    for (int t = 0; t < T; ++t) v[t] = f[j * T + t];
    rdft<T>(v, q);
#pragma unroll
    for (int p = 0; p < T; ++p) P[p][j] = q[p];
  }
}

// fp16: the HKW channels of one lane taken in pairs (2j, 2j+1), element t of
// both in one packed register, and transformed together in fp16 arithmetic;
// W[p][j] is then plane p of the pair, the word that is staged.  Element t of
// channel c is half (c*T + t) % 2 of raw word (c*T + t) / 2.
template <int T, int HKW>
__device__ __forceinline__ void raw_to_packed_planes(const uint32_t (&r)[HKW * T / 2],
                                                     uint32_t (&W)[T][HKW / 2]) {
  static_for<HKW / 2>([&](auto ji) {
    constexpr int j = decltype(ji)::value;
    half2v v[T], P[T];
    static_for<T>([&](auto ti) {
      constexpr int t = decltype(ti)::value;
      constexpr int ia = (2 * j) * T + t, ib = (2 * j + 1) * T + t;
      v[t] = pair_halves<ia % 2, ib % 2>(r[ia / 2], r[ib / 2]);
    });
    rdft<T, H2Ops>(v, P);
#pragma unroll
    for (int p = 0; p < T; ++p) W[p][j] = __builtin_bit_cast(uint32_t, P[p]);
  });
}

}  // namespace eqk

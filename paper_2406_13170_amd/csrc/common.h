// Shared device helpers for the gfx950 kernels: 16-byte fragments of float / bfloat16, the matrix-core
// step on such fragments, and wave / block reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace amph {

typedef __bf16 bf16_t;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int WAVE = 64;
constexpr float NEG_BIG = -1.0e30f;   // finite stand-in for -inf in running maxima

// ---- element traits: PER = elements in one 16-byte fragment ------------------------------------
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int PER = 4;
  static __device__ __forceinline__ void unpack(const uint4 &v, float *f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  static __device__ __forceinline__ float to_f32(float v) { return v; }
  static __device__ __forceinline__ float from_f32(float v) { return v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int PER = 8;
  static __device__ __forceinline__ void unpack(const uint4 &v, float *f) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
  static __device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
  static __device__ __forceinline__ bf16_t from_f32(float v) { return (bf16_t)v; }   // RNE
};

// pack PER floats into one 16-byte fragment of T (RNE for bf16)
template <typename T> __device__ __forceinline__ uint4 pack16(const float *f);
template <> __device__ __forceinline__ uint4 pack16<float>(const float *f) {
  return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
}
template <> __device__ __forceinline__ uint4 pack16<bf16_t>(const float *f) {
  union { bf16x8 v; uint4 u; } c;
  #pragma unroll
  for (int i = 0; i < 8; ++i) c.v[i] = (bf16_t)f[i];
  return c.u;
}

__device__ __forceinline__ uint4 ldg16(const void *p) { return *reinterpret_cast<const uint4 *>(p); }
// the same load marked non-temporal: data that is read once (a weight stream) should not push reused data out of L2
__device__ __forceinline__ uint4 ldg16_stream(const void *p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stg16(void *p, const uint4 &v) { *reinterpret_cast<uint4 *>(p) = v; }

// 4 consecutive elements of T <-> float[4]
template <typename T> __device__ __forceinline__ void load4(const T *p, float *f);
template <> __device__ __forceinline__ void load4<float>(const float *p, float *f) {
  const float4 v = *reinterpret_cast<const float4 *>(p);
  f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
template <> __device__ __forceinline__ void load4<bf16_t>(const bf16_t *p, float *f) {
  const uint2 v = *reinterpret_cast<const uint2 *>(p);
  f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
  f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
}
template <typename T> __device__ __forceinline__ void store4(T *p, const float *f);
template <> __device__ __forceinline__ void store4<float>(float *p, const float *f) {
  *reinterpret_cast<float4 *>(p) = make_float4(f[0], f[1], f[2], f[3]);
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t *p, const float *f) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 v;
  #pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (bf16_t)f[i];
  *reinterpret_cast<bf16x4 *>(p) = v;
}

// ---- matrix-core step on 16-byte fragments --------------------------------------------------------
// D[16 x 16] += A[16 x KS] * B[KS x 16] with KS = 4 * PER.  Lane l holds for A: row l%16, contraction
// slots (l/16)*PER .. +PER; for B: column l%16, the same slots; for D: column l%16, rows (l/16)*4..+4.
// bf16: one 16x16x32 instruction.  float: four 16x16x4 instructions, the j-th using element j of
// every lane's fragment (any one-to-one slot assignment is valid as long as A and B agree).
template <typename T> __device__ __forceinline__ f32x4 mma16(const uint4 &a, const uint4 &b, f32x4 acc);
template <> __device__ __forceinline__ f32x4 mma16<bf16_t>(const uint4 &a, const uint4 &b, f32x4 acc) {
  union { uint4 u; bf16x8 v; } ca, cb;
  ca.u = a; cb.u = b;
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ca.v, cb.v, acc, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma16<float>(const uint4 &a, const uint4 &b, f32x4 acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  return acc;
}

// Element index of (row, dim) in the step-tiled K and V caches of one head (layout: header of the C ABI).
template <typename T> __device__ __forceinline__ size_t k_tiled_index(int row, int c, int d_h) {
  constexpr int PER = Elem<T>::PER, KSTEP = 4 * PER, PIECE = 64 / (int)sizeof(T);   // elements in 64 bytes
  const int s = row / KSTEP, kk = row % KSTEP, t = (kk % PER) / 4, i = (kk / PER) * 4 + (kk & 3);
  return ((size_t)(s * (PER / 4) + t) * (d_h / PIECE) + c / PIECE) * (16 * PIECE) + i * PIECE + c % PIECE;
}
template <typename T> __device__ __forceinline__ size_t v_tiled_index(int row, int c, int d_h) {
  constexpr int PER = Elem<T>::PER, KSTEP = 4 * PER, PIECE = 64 / (int)sizeof(T);
  return ((size_t)(row / KSTEP) * (d_h / 16) + c / 16) * (16 * PIECE) + (c % 16) * PIECE + row % KSTEP;
}

// Element index of (row m, element k) in the fragment-tiled activation layout the wide GEMM reads: 16 rows x 64 bytes
// of k per KB, lane-linear (lane = g * 16 + m % 16 holds the 16 bytes at g * 16), the two fragments of 32 rows side by side.
// 4 elements starting at a multiple of 4 stay inside one 16-byte piece.
template <typename T> __device__ __forceinline__ size_t xt_index(int m, int k, int m32_tiles) {
  const int kb = k * (int)sizeof(T);
  const size_t byte = ((size_t)(kb >> 6) * (2 * m32_tiles) + (m >> 4)) * 1024 + (size_t)((((kb >> 4) & 3) * 16 + (m & 15)) << 4) + (kb & 15);
  return byte / sizeof(T);
}

// ---- wave-level reductions ---------------------------------------------------------------------------
// The 32-bit value of the lane OFF further on, exchanged inside the vector ALU (a shuffle goes through LDS: about a hundred
// clocks of latency each, and its turn there; six of them for every sum were a good part of the short kernels: a whole
// iteration of the float32 miniature 216 -> 203 us; longer kernels do not show it).
// xor16 / xor32: the row swap of a register with itself leaves the even rows (the lower half) in one result and the odd
// ones (the upper half) in the other, so op of the two is op over lanes 16 (32) apart, in every lane.
template <typename V> __device__ __forceinline__ unsigned lane_bits(V v) { union { V v; unsigned u; } c; c.v = v; return c.u; }
template <typename V> __device__ __forceinline__ V lane_value(unsigned u) { union { unsigned u; V v; } c; c.u = u; return c.v; }
template <typename V, typename F> __device__ __forceinline__ V lanes_xor16(V v, F op) {
  const auto p = __builtin_amdgcn_permlane16_swap(lane_bits(v), lane_bits(v), false, false);
  return op(lane_value<V>(p[0]), lane_value<V>(p[1]));
}
template <typename V, typename F> __device__ __forceinline__ V lanes_xor32(V v, F op) {
  const auto p = __builtin_amdgcn_permlane32_swap(lane_bits(v), lane_bits(v), false, false);
  return op(lane_value<V>(p[0]), lane_value<V>(p[1]));
}
template <int CTRL, typename V> __device__ __forceinline__ V lanes_dpp(V v) {
  return lane_value<V>((unsigned)__builtin_amdgcn_update_dpp(0, (int)lane_bits(v), CTRL, 0xf, 0xf, true));
}
template <int N, typename V> __device__ __forceinline__ V lanes_ror(V v) { return lanes_dpp<0x120 + N>(v); }   // rotation inside rows of 16
constexpr int DPP_XOR1 = 0xb1, DPP_XOR2 = 0x4e;           // quad_perm [1, 0, 3, 2] and [2, 3, 0, 1]
// op (commutative) over the 64 lanes, in every lane: partners 32, 16, 8, 4, 2, 1 apart.  Once lanes 2 N apart hold the same
// value, the lane N before in the row is the partner N apart: the order, and so the bits, of a butterfly of shuffles.
// All 64 lanes must be active.
template <typename V, typename F> __device__ __forceinline__ V wave_fold(V v, F op) {
  v = lanes_xor32(v, op);
  v = lanes_xor16(v, op);
  v = op(v, lanes_ror<8>(v));
  v = op(v, lanes_ror<4>(v));
  v = op(v, lanes_ror<2>(v));
  return op(v, lanes_ror<1>(v));
}
struct AddF { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct MaxF { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct MaxI { __device__ __forceinline__ int operator()(int a, int b) const { return max(a, b); } };
__device__ __forceinline__ float wave_sum(float v) { return wave_fold(v, AddF()); }
__device__ __forceinline__ float wave_max(float v) { return wave_fold(v, MaxF()); }
__device__ __forceinline__ int wave_max(int v) { return wave_fold(v, MaxI()); }

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

// ---- selection inside one wave (top-k of Eq. 6) ---------------------------------------------------------
// "Better" means a larger value, or the same value and a smaller index, so results are sorted and ties deterministic.
__device__ __forceinline__ bool better(float v1, int i1, float v2, int i2) {
  return (v1 > v2) || (v1 == v2 && i1 < i2);
}
__device__ __forceinline__ void take_better(float &v, int &i, float ov, int oi) {
  if (better(ov, oi, v, i)) { v = ov; i = oi; }
}
// the best (value, index) of the 64 lanes, in every lane
__device__ __forceinline__ void wave_best(float &v, int &i) {
  const auto pv = __builtin_amdgcn_permlane32_swap(lane_bits(v), lane_bits(v), false, false);
  const auto pi = __builtin_amdgcn_permlane32_swap(lane_bits(i), lane_bits(i), false, false);
  v = lane_value<float>(pv[0]); i = (int)pi[0];
  take_better(v, i, lane_value<float>(pv[1]), (int)pi[1]);
  const auto qv = __builtin_amdgcn_permlane16_swap(lane_bits(v), lane_bits(v), false, false);
  const auto qi = __builtin_amdgcn_permlane16_swap(lane_bits(i), lane_bits(i), false, false);
  v = lane_value<float>(qv[0]); i = (int)qi[0];
  take_better(v, i, lane_value<float>(qv[1]), (int)qi[1]);
  take_better(v, i, lanes_ror<8>(v), lanes_ror<8>(i));
  take_better(v, i, lanes_ror<4>(v), lanes_ror<4>(i));
  take_better(v, i, lanes_ror<2>(v), lanes_ror<2>(i));
  take_better(v, i, lanes_ror<1>(v), lanes_ror<1>(i));
}

// Selection by counting: an element's place among the best is the number of better ones, which every lane counts for its
// own elements against all of them, one broadcast at a time.  The k places come out at once.  (In k rounds of a wave-wide
// maximum, each a chain of six cross-lane steps and a rescan of about 1000 clocks, ten places among 64 logits made the
// LM head's epilogue 4 us long; this takes less than one round did.)
// Order-preserving integer of a float, at least 1; 0 for NaN (never selected).  +0 and -0 are equal.
__device__ __forceinline__ unsigned rank_key(float v) {
  const unsigned b = __float_as_uint(v + 0.0f);
  return (v == v) ? b ^ (((int)b < 0) ? 0xffffffffu : 0x80000000u) : 0u;
}
// number of the NPT * 64 keys (element j * 64 + lane; 0 = none) that come before own key at place own_e: larger, or equal
// at a lower place.  Elements from n on are not looked at.  All 64 lanes must be active.
template <int NPT>
__device__ __forceinline__ int rank_among(const unsigned (&key)[NPT], int n, unsigned own, int own_e) {
  int rank = 0;
  #pragma unroll
  for (int j = 0; j < NPT; ++j) {
    if (j * WAVE < n) {
      #pragma unroll 8
      for (int s = 0; s < WAVE; ++s) {                     // (unrolled whole, the broadcast values fill the scalar registers)
        const unsigned o = (unsigned)__builtin_amdgcn_readlane((int)key[j], s);
        rank += (o > own || (o == own && j * WAVE + s < own_e)) ? 1 : 0;
      }
    }
  }
  return rank;
}
// The k best of NPT values per lane (element e = j * 64 + lane, token id0 + e, e < n_live) into out_v / out_i, best first, ties
// to the lower token; (-inf, -1) past the last one.
template <int NPT>
__device__ __forceinline__ void rank_select(const float (&x)[NPT], int id0, int n_live, int k, float *out_v, int *out_i) {
  const int lane = threadIdx.x & 63;
  unsigned key[NPT];
  int n_valid = 0;
  #pragma unroll
  for (int j = 0; j < NPT; ++j) {
    key[j] = (j * WAVE + lane < n_live) ? rank_key(x[j]) : 0u;
    n_valid += __popcll(__ballot(key[j] != 0u));
  }
  #pragma unroll
  for (int j = 0; j < NPT; ++j) {
    const int r = rank_among<NPT>(key, n_live, key[j], j * WAVE + lane);
    if (key[j] != 0u && r < k) { out_v[r] = x[j]; out_i[r] = id0 + j * WAVE + lane; }
  }
  if (lane >= n_valid && lane < k) { out_v[lane] = -__builtin_huge_valf(); out_i[lane] = -1; }
}

}  // namespace amph

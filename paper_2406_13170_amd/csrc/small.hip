// The small kernels of the step: single-query attention of the adaptation layers over their caches
// (Eq. 1), the K x K bi-directional attention of Eq. 5, per-row top-k / argmax (Eq. 6), candidate-tree
// construction, greedy acceptance, and the row-wise RMSNorm (+ partial-sum fold) of the target path.
#include "kernels.h"
#include <algorithm>

namespace amph {

// =====================================================================================================
// Attention of the adaptation layers over their caches: query row (b, j) = new position j of batch element b against
// rows [0, sal_len[b] + j] of the cache (its own new row included, later new rows excluded: causal among the new
// positions).  A stream of the caches with little arithmetic, so what counts is that every row is read once and that
// enough compute units read:
//   * a workgroup serves up to RT new positions of a (head, batch element) together, from the same key and value
//     fragments (one workgroup per position read the cache R times: 33B widths, batch 4, 6 positions, 2047 rows 99 us,
//     now 58; 7B, batch 8, 5 positions 40 us, now 32);
//   * with few heads the cache rows are split over S workgroups, whose (max, sum, weighted values) k_sal_fold merges in
//     ascending order (7B, batch 1, 1024 rows, one workgroup per head 15.8 us, now 6.1 + 4.7 us).
// grid = (heads, batch * row groups, S), 512 threads: the 8 waves stride over the rows.  Each 16-byte fragment of a
// key/value row belongs to one lane; LPR lanes share a row, so a wave covers 64 / LPR rows per load.  Running (max, sum,
// weighted values) are merged lane group -> wave -> workgroup.
// kv_stage: [B, 2, n_heads, max_kv, DH] T.   out: [rows, d] float32.
// =====================================================================================================
constexpr int SA_WAVES = 8;

// 2^x by the hardware instruction alone: arguments here are at most 0, and what would be below the normal range may be 0
__device__ __forceinline__ float sa_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <bool V> struct BoolTag { static constexpr bool value = V; };
// sum over groups of LPR adjacent lanes, in every lane: neighbour at distance 1, 2, then mirror inside 8 and inside 16
// lanes, each one vector instruction (a cross-lane permute goes through LDS)
template <int LPR> __device__ __forceinline__ float sa_group_sum(float v) {
  #define SA_DPP(CTRL) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true))
  SA_DPP(0xb1);                          // quad_perm [1, 0, 3, 2]
  SA_DPP(0x4e);                          // quad_perm [2, 3, 0, 1]
  if (LPR >= 8) SA_DPP(0x141);           // row_half_mirror
  if (LPR >= 16) SA_DPP(0x140);          // row_mirror
  #undef SA_DPP
  if (LPR >= 32) v = lanes_xor16(v, AddF());
  return v;
}
// op over the lane groups of LPR lanes (the same lane of each), in every lane
template <int LPR, typename F> __device__ __forceinline__ float sa_across(float v, F op) {
  if (LPR <= 8) v = op(v, lanes_ror<8>(v));
  if (LPR <= 16) v = lanes_xor16(v, op);
  return lanes_xor32(v, op);
}

template <typename T, int DH, int RT>
__global__ __launch_bounds__(SA_WAVES * 64) void k_sal_attn(const float *qbuf, const T *kv_stage, const int32_t *sal_len,
                                                            int n_heads, int max_kv, float *out, int R,
                                                            const int32_t *n_valid, int last_only, int n_groups, float *part) {
  constexpr int PER = Elem<T>::PER;
  constexpr int LPR = DH / PER;          // lanes per row
  constexpr int G = WAVE / LPR;          // rows per wave load
  constexpr int U = 4;
  __shared__ float sm_m[SA_WAVES][RT], sm_l[SA_WAVES][RT];
  __shared__ float sm_o[SA_WAVES][RT][DH];
  // last_only: one row per batch element, its last live position (query row b * R + jn of qbuf, output row b);
  // otherwise rows j0 .. j0 + RT - 1 of the element
  const int h = blockIdx.x, b = blockIdx.y / n_groups, j0 = (blockIdx.y % n_groups) * RT;
  const int S = gridDim.z, split = blockIdx.z;
  const int d = n_heads * DH;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = lane / LPR, li = lane % LPR;
  const int sl = sal_len[b], nv = n_valid ? n_valid[b] : R;
  int n[RT], n_max = 0, n_all = 0x7fffffff;               // rows of the cache that each query sees (0: dead); rows that all live ones see
  float qv[RT][PER];
  const float scale = 1.4426950408889634f * rsqrtf((float)DH);
  #pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int jn = last_only ? min(max(nv, 1), R) - 1 : j0 + r;
    const bool live = jn < R && !(n_valid && jn >= nv);
    n[r] = (!live || sl < 0 || sl + jn + 1 > max_kv) ? 0 : sl + jn + 1;
    n_max = max(n_max, n[r]);
    if (n[r] > 0) n_all = min(n_all, n[r]);
    const float *q = qbuf + (size_t)(b * R + min(jn, R - 1)) * d + h * DH + li * PER;
    #pragma unroll
    for (int j = 0; j < PER; ++j) qv[r][j] = q[j] * scale;
  }
  const T *kbase = kv_stage + (((size_t)b * 2 + 0) * n_heads + h) * (size_t)max_kv * DH;
  const T *vbase = kv_stage + (((size_t)b * 2 + 1) * n_heads + h) * (size_t)max_kv * DH;
  float m[RT], l[RT], o[RT][PER];
  #pragma unroll
  for (int r = 0; r < RT; ++r) {
    m[r] = NEG_BIG; l[r] = 0.f;
    #pragma unroll
    for (int j = 0; j < PER; ++j) o[r][j] = 0.f;
  }
  const int per = (n_max + S - 1) / S, k0 = split * per, k1 = min(k0 + per, n_max);
  // U rows per lane group against all queries: scores, one move of the running maxima, probabilities, values.  MASKED:
  // some of the rows lie past the range or are hidden from some query (the last batch of a range only).
  auto batch = [&](auto tag, int jb, const uint4 (&kf)[U], const uint4 (&vf)[U]) {
    constexpr bool MASKED = decltype(tag)::value;
    float sc[RT][U];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
      float kk[PER];
      Elem<T>::unpack(kf[u], kk);
      const int j = jb + u * G + grp;
      #pragma unroll
      for (int r = 0; r < RT; ++r) {
        float s = 0.f;
        #pragma unroll
        for (int e = 0; e < PER; ++e) s = fmaf(qv[r][e], kk[e], s);
        s = sa_group_sum<LPR>(s);
        sc[r][u] = (MASKED && !(j < k1 && j < n[r])) ? -__builtin_huge_valf() : s;
      }
    }
    #pragma unroll
    for (int r = 0; r < RT; ++r) {
      float mn = m[r];
      #pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, sc[r][u]);
      const float corr = sa_exp2(m[r] - mn);               // (mn is at least NEG_BIG: masked scores give 2^-inf = 0)
      m[r] = mn;
      l[r] *= corr;
      #pragma unroll
      for (int e = 0; e < PER; ++e) o[r][e] *= corr;
      #pragma unroll
      for (int u = 0; u < U; ++u) { sc[r][u] = sa_exp2(sc[r][u] - mn); l[r] += sc[r][u]; }
    }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
      float vv[PER];
      Elem<T>::unpack(vf[u], vv);
      const int j = jb + u * G + grp;
      #pragma unroll
      for (int r = 0; r < RT; ++r) {
        const bool in = !MASKED || (j < k1 && j < n[r]);   // a hidden row is left out whatever it holds (0 * NaN)
        #pragma unroll
        for (int e = 0; e < PER; ++e) o[r][e] = in ? fmaf(sc[r][u], vv[e], o[r][e]) : o[r][e];
      }
    }
  };
  for (int jb = k0 + wave * (U * G); jb < k1; jb += SA_WAVES * U * G) {
    uint4 kf[U], vf[U];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(jb + u * G + grp, k1 - 1);         // unconditional loads; rows past the end are masked
      kf[u] = ldg16_stream(kbase + (size_t)j * DH + li * PER);
      vf[u] = ldg16_stream(vbase + (size_t)j * DH + li * PER);
    }
    if (jb + U * G <= min(k1, n_all)) batch(BoolTag<false>{}, jb, kf, vf);        // (uniform over the wave)
    else batch(BoolTag<true>{}, jb, kf, vf);
  }
  #pragma unroll
  for (int r = 0; r < RT; ++r)
    if (n[r] == 0) { m[r] = NEG_BIG; l[r] = 0.f; }         // a dead position (its output is zero)
  // lane groups -> wave
  #pragma unroll
  for (int r = 0; r < RT; ++r) {
    const float mw = sa_across<LPR>(m[r], MaxF());
    const float f = sa_exp2(m[r] - mw);
    m[r] = mw;
    l[r] = sa_across<LPR>(l[r] * f, AddF());
    #pragma unroll
    for (int e = 0; e < PER; ++e) o[r][e] = sa_across<LPR>(o[r][e] * f, AddF());
    if (grp == 0) {
      #pragma unroll
      for (int e = 0; e < PER; ++e) sm_o[wave][r][li * PER + e] = o[r][e];
      if (li == 0) { sm_m[wave][r] = m[r]; sm_l[wave][r] = l[r]; }
    }
  }
  __syncthreads();
  // waves -> workgroup
  for (int idx = threadIdx.x; idx < RT * DH; idx += SA_WAVES * 64) {
    const int r = idx / DH, e = idx % DH;
    if (!last_only && j0 + r >= R) break;
    const int row = last_only ? b : b * R + j0 + r;
    float mw = sm_m[0][r];
    #pragma unroll
    for (int w = 1; w < SA_WAVES; ++w) mw = fmaxf(mw, sm_m[w][r]);
    float lw = 0.f, ow = 0.f;
    #pragma unroll
    for (int w = 0; w < SA_WAVES; ++w) {
      const float f = sa_exp2(sm_m[w][r] - mw);
      lw += sm_l[w][r] * f;
      ow += sm_o[w][r][e] * f;
    }
    if (S == 1) {
      out[(size_t)row * d + h * DH + e] = (lw > 0.f) ? ow / lw : 0.f;
    } else {
      float *p = part + (((size_t)row * n_heads + h) * S + split) * sal_part_pitch(DH);
      p[e] = ow;
      if (e == 0) { p[DH] = mw; p[DH + 1] = lw; }
    }
  }
}

// out[row] of one head = sum_s o_s 2^(m_s - m) / sum_s l_s 2^(m_s - m), s ascending; every split's values are requested
// before the first is used.  grid = (heads, rows), DH threads.
template <int DH>
__global__ __launch_bounds__(DH) void k_sal_fold(const float *part, int n_heads, int S, float *out) {
  const int h = blockIdx.x, row = blockIdx.y, e = threadIdx.x;
  const float *p = part + ((size_t)row * n_heads + h) * S * sal_part_pitch(DH);
  float ov[SAL_MAX_SPLITS], mv[SAL_MAX_SPLITS], lv[SAL_MAX_SPLITS];
  #pragma unroll
  for (int s = 0; s < SAL_MAX_SPLITS; ++s) {
    const float *ps = p + (size_t)min(s, S - 1) * sal_part_pitch(DH);
    ov[s] = ps[e]; mv[s] = ps[DH]; lv[s] = ps[DH + 1];
  }
  float mw = NEG_BIG;
  #pragma unroll
  for (int s = 0; s < SAL_MAX_SPLITS; ++s) if (s < S) mw = fmaxf(mw, mv[s]);
  float lw = 0.f, ow = 0.f;
  #pragma unroll
  for (int s = 0; s < SAL_MAX_SPLITS; ++s)
    if (s < S) {
      const float f = exp2f(mv[s] - mw);
      lw += lv[s] * f;
      ow += ov[s] * f;
    }
  out[((size_t)row * n_heads + h) * DH + e] = (lw > 0.f) ? ow / lw : 0.f;
}

// New positions per workgroup: one where that leaves fewer workgroups than compute units (their caches then come from L2
// for all but the first, and six queries' arithmetic would be the longest part: 32 heads, 5 positions, 1024 rows: five
// workgroups per head 15.1 us, one with 8 key splits 11.8 + 4.8 for the fold), else as many as go together.
static int sal_group(int B, int n_heads, int R) { return (R <= 1 || B * n_heads * R <= 256) ? 1 : R <= 3 ? 3 : 6; }
// Key splits, of 128 rows or more, where they pay for the fold: one workgroup per compute unit, of the small
// ones (one position) two, from five splits on (one position, 208 workgroups of 2047 rows: 33.8 us whole, 35.6 + 4.9 in
// two splits; 160 of 1024 rows 15.1, 11.2 + 4.9 in three; 32 of 1024 rows 15.8, 6.1 + 4.7 in eight).  The lengths are the
// device's, so the rule reads the capacity, and a short context in a large cache pays for splits that it does not need
// (whole drafts of one position, caches of 4096 rows, us whole / split: 7B, 100 rows 357 / 363, 600 367 / 367, 1000
// 375 / 370, 4000 427 / 383; the float32 miniature 95 / 96, 106 / 99, 112 / 101, 164 / 109).
static int sal_splits(int B, int n_groups, int n_heads, int max_kv, int rt) {
  const int s = std::min((rt == 1 ? 480 : 256) / (B * n_groups * n_heads), max_kv / 128);
  return (rt == 1 && s < 5) ? 1 : std::max(1, std::min(s, SAL_MAX_SPLITS));
}
int sal_key_splits(int B, int R, int last_only, int n_heads, int max_kv) {
  const int rt = last_only ? 1 : sal_group(B, n_heads, R), n_groups = last_only ? 1 : (R + rt - 1) / rt;
  return sal_splits(B, n_groups, n_heads, max_kv, rt);
}
size_t sal_part_floats(int B, int R, int n_heads, int d_h, int max_kv) {
  size_t most = 0;
  for (int r = 1; r <= R; ++r) {                            // any number of new positions up to R may be asked for
    const int rt = sal_group(B, n_heads, r), s = sal_splits(B, (r + rt - 1) / rt, n_heads, max_kv, rt);
    if (s > 1) most = std::max(most, (size_t)B * r * n_heads * s * sal_part_pitch(d_h));
  }
  return most;
}

template <typename T, int DH>
static hipError_t launch_sal_attn_dh(hipStream_t st, const float *qbuf, const T *kv_stage, const int32_t *sal_len, int B, int n_heads,
                                     int max_kv, float *out, int R, const int32_t *n_valid, int last_only, float *part, bool fold) {
  const int rt = last_only ? 1 : sal_group(B, n_heads, R), n_groups = last_only ? 1 : (R + rt - 1) / rt;
  const int S = sal_key_splits(B, R, last_only, n_heads, max_kv);
  const dim3 grid(n_heads, B * n_groups, S), block(SA_WAVES * 64);
  #define SA(RT_) hipLaunchKernelGGL((k_sal_attn<T, DH, RT_>), grid, block, 0, st, qbuf, kv_stage, sal_len, n_heads, max_kv, out, R, n_valid, \
                                     last_only, n_groups, part)
  if (rt == 1) SA(1); else if (rt == 3) SA(3); else SA(6);
  #undef SA
  if (S > 1 && fold) hipLaunchKernelGGL((k_sal_fold<DH>), dim3(n_heads, last_only ? B : B * R), dim3(DH), 0, st, part, n_heads, S, out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sal_attn(hipStream_t st, const float *qbuf, const void *kv_stage, const int32_t *sal_len, int B,
                           int n_heads, int d_h, int max_kv, float *out, int R, const int32_t *n_valid, int last_only, float *part, bool fold) {
  if (d_h == 64) return launch_sal_attn_dh<T, 64>(st, qbuf, (const T *)kv_stage, sal_len, B, n_heads, max_kv, out, R, n_valid, last_only, part, fold);
  if (d_h == 128) return launch_sal_attn_dh<T, 128>(st, qbuf, (const T *)kv_stage, sal_len, B, n_heads, max_kv, out, R, n_valid, last_only, part, fold);
  return hipErrorInvalidValue;
}
template hipError_t launch_sal_attn<float>(hipStream_t, const float *, const void *, const int32_t *, int, int, int, int,
                                           float *, int, const int32_t *, int, float *, bool);
template hipError_t launch_sal_attn<bf16_t>(hipStream_t, const float *, const void *, const int32_t *, int, int, int,
                                            int, float *, int, const int32_t *, int, float *, bool);

// =====================================================================================================
// Eq. 5 core: for one (batch, head) the K x K score matrix of the K head positions, a row softmax
// with no mask, and the weighted sum of the value rows.  Q, Kk, V, ctx: [B * K, d] float32.
// The head's K rows of Q, K and V are first parked in LDS.
// =====================================================================================================
__global__ __launch_bounds__(128) void k_aeb_attn(const float *Q, const float *Kk, const float *V, int K, int n_heads,
                                                  int d_h, float *ctx) {
  __shared__ float sq[AMPH_MAX_HEADS_K * 128], sk[AMPH_MAX_HEADS_K * 128], sv[AMPH_MAX_HEADS_K * 128];
  __shared__ float sc[AMPH_MAX_HEADS_K * AMPH_MAX_HEADS_K];
  const int h = blockIdx.x, b = blockIdx.y;
  const int d = n_heads * d_h;
  const size_t base = (size_t)b * K * d + (size_t)h * d_h;
  const int t = threadIdx.x;
  for (int i = t; i < K * d_h; i += blockDim.x) {
    const int r = i / d_h, e = i % d_h;
    sq[i] = Q[base + (size_t)r * d + e];
    sk[i] = Kk[base + (size_t)r * d + e];
    sv[i] = V[base + (size_t)r * d + e];
  }
  __syncthreads();
  if (t < K * K) {
    const int i = t / K, j = t % K;
    float s = 0.f;
    for (int e = 0; e < d_h; ++e) s = fmaf(sq[i * d_h + e], sk[j * d_h + e], s);
    sc[t] = s * rsqrtf((float)d_h);
  }
  __syncthreads();
  if (t < K) {
    float mx = sc[t * K];
    for (int j = 1; j < K; ++j) mx = fmaxf(mx, sc[t * K + j]);
    float sum = 0.f;
    for (int j = 0; j < K; ++j) { const float e = __expf(sc[t * K + j] - mx); sc[t * K + j] = e; sum += e; }
    const float inv = 1.0f / sum;
    for (int j = 0; j < K; ++j) sc[t * K + j] *= inv;
  }
  __syncthreads();
  for (int e = t; e < d_h; e += blockDim.x) {
    for (int i = 0; i < K; ++i) {
      float o = 0.f;
      for (int j = 0; j < K; ++j) o = fmaf(sc[i * K + j], sv[j * d_h + e], o);
      ctx[base + (size_t)i * d + e] = o;
    }
  }
}

hipError_t launch_aeb_attn(hipStream_t st, const float *Q, const float *Kk, const float *V, int B, int K, int n_heads,
                           int d_h, float *ctx) {
  if (K < 1 || K > AMPH_MAX_HEADS_K || d_h > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_aeb_attn, dim3(n_heads, B), dim3(128), 0, st, Q, Kk, V, K, n_heads, d_h, ctx);
  return hipGetLastError();
}

// =====================================================================================================
// Top-k of the draft's rows (Eq. 6) and argmax of the target's.  "Better" means a larger value, or the same value and a
// smaller index, so results are sorted and ties deterministic.
// =====================================================================================================
// Cache length of element i after its new rows: advanced only when every new row fitted (the kernels that write
// the rows skipped those past the limit and raised the overflow flag; the length then stays where it was).
__device__ __forceinline__ void advance_one(int32_t *len, int i, int by, int limit) {
  const int v = len[i];
  if (v >= 0 && by >= 0 && v + by <= limit) len[i] = v + by;
}

// Top-k of the candidates the fused LM head left: per row n_lists lists of k (value, token) pairs, each sorted (best
// first, token -1 past its end), the lists in ascending token order.  One workgroup per row, three selections by counting
// the better ones:
//   1. every wave takes the k best heads of 64 lists;
//   2. of those the k best heads of all (ties to the lower list, which holds the lower tokens): a list whose head is not
//      among them has k better candidates elsewhere;
//   3. the k best of those lists' k * k candidates.
// (Sixteen waves selecting in rounds over all 5000 candidates of 500 lists: 14.6 us, one wave in rounds over the heads and
// then the chosen lists 13.7, this 7.9; a launch that loads, loads what that names and stores is 4.8.)
template <int W>
__global__ __launch_bounds__(W * 64) void k_topk_merge(const float *cand_v, const int *cand_i, int n_lists, int V, int k,
                                                       int32_t *idx, float *val, int32_t *advance, int n_advance, int advance_by,
                                                       const int32_t *advance_each, int advance_limit) {
  constexpr int MK = AMPH_MAX_TOPK;
  static_assert(W * 64 >= MK * MK, "one thread per candidate of the chosen lists");
  __shared__ float hv[W * MK];
  __shared__ int hi[W * MK], sel[MK];
  __shared__ unsigned long long key[W * 64];
  const int row = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float *cv = cand_v + (size_t)row * n_lists * k;
  const int *ci = cand_i + (size_t)row * n_lists * k;
  // a key of its own for every (value, id): larger is better, ties to the lower id; 0 = none
  auto key_of = [](float v, int id) {
    const unsigned q = rank_key(v);
    return (id >= 0 && q != 0u) ? ((unsigned long long)q << 32) | (unsigned)~id : 0ull;
  };
  auto place = [&](unsigned long long own, int n) {
    int r = 0;
    for (int e = 0; e < n; ++e) r += key[e] > own ? 1 : 0;
    return r;
  };
  {
    const int li = tid, lc = min(li, n_lists - 1), t = ci[(size_t)lc * k];
    float x[1] = {cv[(size_t)lc * k]};
    if (t < 0 || t >= V) x[0] = __builtin_nanf("");        // no candidate
    rank_select<1>(x, wave * WAVE, min(max(n_lists - wave * WAVE, 0), WAVE), k, hv + wave * k, hi + wave * k);
  }
  if (tid < k) sel[tid] = -1;
  __syncthreads();
  unsigned long long own = 0ull;
  if (tid < W * k) key[tid] = own = key_of(hv[tid], hi[tid]);
  __syncthreads();
  if (own != 0ull) {
    const int r = place(own, W * k);
    if (r < k) sel[r] = hi[tid];
  }
  __syncthreads();
  const int list = tid < k * k ? sel[tid / k] : -1;
  float y = 0.f;
  int tk = -1;
  if (list >= 0) {
    y = cv[(size_t)list * k + tid % k];
    tk = ci[(size_t)list * k + tid % k];
  }
  own = key_of(y, tk < V ? tk : -1);
  key[tid] = own;
  const int n_valid = __syncthreads_count(own != 0ull);
  if (own != 0ull) {
    const int r = place(own, k * k);
    if (r < k) {
      if (idx) idx[(size_t)row * k + r] = tk;
      if (val) val[(size_t)row * k + r] = y;
    }
  }
  if (tid >= n_valid && tid < k) {
    if (idx) idx[(size_t)row * k + tid] = -1;
    if (val) val[(size_t)row * k + tid] = -__builtin_huge_valf();
  }
  if (row == 0 && advance)
    for (int i = tid; i < n_advance; i += W * 64) advance_one(advance, i, advance_each ? advance_each[i] : advance_by, advance_limit);
}

hipError_t launch_topk_merge(hipStream_t st, const float *cand_v, const int *cand_i, int rows, int n_cand, int V, int k,
                             int32_t *idx, float *val, int32_t *advance, int n_advance, int advance_by,
                             const int32_t *advance_each, int advance_limit) {
  if (rows < 1 || n_cand < 1 || k < 1 || k > AMPH_MAX_TOPK || n_cand % k || n_cand / k > LMTK_MAX_WG) return hipErrorInvalidValue;
  const int n_lists = n_cand / k;
  #define TM_LAUNCH(W) hipLaunchKernelGGL((k_topk_merge<W>), dim3(rows), dim3(W * 64), 0, st, cand_v, cand_i, n_lists, V, k, idx, val, \
                                          advance, n_advance, advance_by, advance_each, advance_limit)
  if (n_lists <= 4 * WAVE) TM_LAUNCH(4); else if (n_lists <= 8 * WAVE) TM_LAUNCH(8); else TM_LAUNCH(16);
  #undef TM_LAUNCH
  return hipGetLastError();
}

// Argmax of a row of up to 65536 logits (amph_accept with logits): 1024 threads, each the best of its NPT logits (all requested
// before the first is used; element j * 1024 + tid in slot j), folded in the wave and through LDS.  -1 if there are only NaN.
template <int NPT>
__global__ __launch_bounds__(1024) void k_row_argmax(const float *logits, int V, int32_t *out) {
  __shared__ float sm_v[16];
  __shared__ int sm_i[16];
  const int NONE = 0x7fffffff;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float *src = logits + (size_t)row * V;
  float x[NPT];
  #pragma unroll
  for (int j = 0; j < NPT; ++j) x[j] = src[min(j * 1024 + tid, V - 1)];        // unconditional loads from clamped addresses
  float bv = -__builtin_huge_valf(); int bi = NONE;
  #pragma unroll
  for (int j = 0; j < NPT; ++j)
    if (j * 1024 + tid < V && better(x[j], j * 1024 + tid, bv, bi)) { bv = x[j]; bi = j * 1024 + tid; }
  wave_best(bv, bi);
  if (lane == 0) { sm_v[wave] = bv; sm_i[wave] = bi; }
  __syncthreads();
  if (wave > 0) return;
  bv = sm_v[lane & 15]; bi = sm_i[lane & 15];
  wave_best(bv, bi);
  if (lane == 0) out[row] = (bi == NONE) ? -1 : bi;
}

hipError_t launch_row_argmax(hipStream_t st, const float *logits, int rows, int V, int32_t *out) {
  if (rows < 1 || V < 1 || V > 65536) return hipErrorInvalidValue;
  #define ROW_ARGMAX(N) hipLaunchKernelGGL((k_row_argmax<N>), dim3(rows), dim3(1024), 0, st, logits, V, out)
  if (V <= 8192) ROW_ARGMAX(8); else if (V <= 16384) ROW_ARGMAX(16); else if (V <= 32768) ROW_ARGMAX(32); else ROW_ARGMAX(64);
  #undef ROW_ARGMAX
  return hipGetLastError();
}

// =====================================================================================================
// Candidate tree: node i at depth m >= 1 takes the rank_i-th candidate of head m; the root takes the
// token the target just sampled; position = committed length + depth.
// =====================================================================================================
__global__ void k_tree_build(const int32_t *depth, const int32_t *rank, int T, int K, int topk,
                             const int32_t *root_tok, const int32_t *topk_idx, const int32_t *kv_len, int32_t *tree_tok,
                             int32_t *tree_pos) {
  const int b = blockIdx.x, i = threadIdx.x;
  if (i >= T) return;
  const int m = depth[i];
  const int tok = (m == 0) ? root_tok[b] : topk_idx[((size_t)b * K + (m - 1)) * topk + rank[i]];
  tree_tok[(size_t)b * T + i] = tok;
  tree_pos[(size_t)b * T + i] = kv_len[b] + m;
}

hipError_t launch_tree_build(hipStream_t st, const int32_t *depth, const int32_t *rank, int T, int B, int K, int topk,
                             const int32_t *root_tok, const int32_t *topk_idx, const int32_t *kv_len, int32_t *tree_tok,
                             int32_t *tree_pos) {
  hipLaunchKernelGGL(k_tree_build, dim3(B), dim3(AMPH_MAX_TREE), 0, st, depth, rank, T, K, topk, root_tok, topk_idx,
                     kv_len, tree_tok, tree_pos);
  return hipGetLastError();
}

// =====================================================================================================
// Greedy acceptance.  Thread i checks its whole ancestor chain (at most K hops): node i is accepted
// iff every node j on the chain carries the target's argmax at parent(j).  The deepest accepted node
// wins (lowest id among equals); thread 0 writes the path by walking up from it.
// =====================================================================================================
__global__ __launch_bounds__(AMPH_MAX_TREE) void k_accept(const int32_t *parent, const int32_t *depth, int T, int K,
                                                          const int32_t *tree_tok, const int32_t *tgt, int32_t *accept_len,
                                                          int32_t *accept_path, int32_t *next_tok, int32_t *best_node) {
  __shared__ int s_key[AMPH_MAX_TREE / WAVE];
  const int b = blockIdx.x, i = threadIdx.x;
  const int32_t *tok = tree_tok + (size_t)b * T;
  const int32_t *tg = tgt + (size_t)b * T;
  int key = -1;
  if (i < T) {
    bool ok = true;
    int j = i;
    for (int hop = 0; hop < AMPH_MAX_HEADS_K && j > 0; ++hop) {
      const int p = parent[j];
      if (tok[j] != tg[p]) { ok = false; break; }
      j = p;
    }
    if (ok) key = depth[i] * 256 + (255 - i);
  }
  key = wave_max(key);
  if ((i & 63) == 0) s_key[i >> 6] = key;
  __syncthreads();
  if (i == 0) {
    int best_key = s_key[0];
    for (int w = 1; w < AMPH_MAX_TREE / WAVE; ++w) best_key = max(best_key, s_key[w]);
    const int a = best_key >> 8, best = 255 - (best_key & 255);     // the root always qualifies
    accept_len[b] = a;
    best_node[b] = best;
    next_tok[b] = tg[best];
    for (int dd = 0; dd <= K; ++dd) accept_path[(size_t)b * (K + 1) + dd] = -1;
    int j = best;
    for (int dd = a; dd >= 0 && j >= 0; --dd) { accept_path[(size_t)b * (K + 1) + dd] = j; j = parent[j]; }
  }
}

hipError_t launch_accept(hipStream_t st, const int32_t *parent, const int32_t *depth, int T, int B, int K,
                         const int32_t *tree_tok, const int32_t *tgt, int32_t *accept_len, int32_t *accept_path,
                         int32_t *next_tok, int32_t *best_node) {
  hipLaunchKernelGGL(k_accept, dim3(B), dim3(AMPH_MAX_TREE), 0, st, parent, depth, T, K, tree_tok, tgt, accept_len,
                     accept_path, next_tok, best_node);
  return hipGetLastError();
}

// =====================================================================================================
// Acceptance under random sampling (Table 2, Temperature = 0.7).  The paper states no rule; the one built is
// typical acceptance as the multi-head framework the paper adopts its tree from defines it: with
// p_j = softmax(logits_j / temperature) and H its entropy in nats, child i of j passes iff
// p_j(tok_i) > min(eps, delta * exp(-H(p_j))); the deepest node whose whole chain passes wins (lowest id among
// equals) and the following token is drawn from p_best by inverting its cumulative distribution (vocabulary
// order) at the caller's uniform number.
//   k_row_softmax_stats: one workgroup per tree node: m = max l, Z = sum exp((l - m) / t),
//     H = ln Z - sum(e x) / Z with x = (l - m) / t, e = exp(x)            -> stats[row] = (m, Z, H, 0)
//     and the row's 1024 run sums (run r: the e of C = ceil(V / 1024) consecutive tokens, added in order) -> runs[row]
//   k_accept_typical: one workgroup per batch element: the pass flags, the winner as in k_accept, then the draw:
//     a scan over the winner's run sums finds the run where the cumulative sum first exceeds u * Z, and one wave
//     walks that run's tokens.  If rounding leaves no such token (u * Z at or above the total), the last token of
//     non-zero probability is taken.
// =====================================================================================================
constexpr int AT_THREADS = 1024, AT_WAVES = AT_THREADS / WAVE;
constexpr int AT_PIECE = 32;                             // logits of a thread whose exponentials sit in LDS at a time
constexpr int AT_MAX_RUN = 64;                           // tokens of a run, at most: one lane each

__device__ __forceinline__ float at_block_max(float v, float *sm) {
  v = wave_max(v);
  __syncthreads();                                        // sm may still be read from an earlier reduction
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sm[0];
  for (int w = 1; w < AT_WAVES; ++w) r = fmaxf(r, sm[w]);
  return r;
}

// A row is read once: its NPT * 1024 logits are all requested before the first is used and stay in registers between the
// maximum and the sums (two strided loops over memory took 23.5 us for 256 rows of 32000; the rows' 33 MB are 7 us).
// Then it is the exponentials that last, 20 vector instructions for each of 32 elements of 16 waves: 5 us of a compute
// unit.  So the draw does not take them again: the run sums leave from here, over LDS, where a thread's elements (t,
// t + 1024, ...) and its run (t C, t C + 1, ...) are different tokens.  That is 1.3 us here for all rows, and 5 us less in
// k_accept_typical, whose one workgroup a sequence fetched a whole row and took its exponentials.
template <int NPT>
__global__ __launch_bounds__(AT_THREADS) void k_row_softmax_stats(const float *logits, int V, float inv_temp, float4 *stats, float *runs) {
  constexpr int PIECE = NPT < AT_PIECE ? NPT : AT_PIECE;
  __shared__ float sm[AT_WAVES], sm2[AT_WAVES];
  __shared__ float s_e[PIECE * AT_THREADS / 32 * 33];      // token v of the piece at v + v / 32: few lanes of a walk meet in one bank
  const float *l = logits + (size_t)blockIdx.x * V;
  const int t = threadIdx.x;
  float x[NPT];
  #pragma unroll
  for (int j = 0; j < NPT; ++j) x[j] = l[min(j * AT_THREADS + t, V - 1)];          // unconditional loads from clamped addresses
  float m = -__builtin_huge_valf();
  #pragma unroll
  for (int j = 0; j < NPT; ++j) m = fmaxf(m, x[j]);       // (the clamped repeats change no maximum)
  m = at_block_max(m, sm);
  const int C = (V + AT_THREADS - 1) / AT_THREADS, v0 = min(t * C, V), v1 = min(v0 + C, V);      // this thread's run
  float z = 0.f, sx = 0.f, run = 0.f;
  #pragma unroll
  for (int p = 0; p < NPT; p += PIECE) {
    if (p > 0) __syncthreads();
    #pragma unroll
    for (int j = 0; j < PIECE; ++j) {
      const int i = j * AT_THREADS + t, v = p * AT_THREADS + i;
      // straight-line code: a repeat past the row's end is a token of probability zero, and such a token adds nothing
      // to sum(e y) (0 * -infinity)
      const float y = v < V ? (x[p + j] - m) * inv_temp : -__builtin_huge_valf(), e = expf(y);
      z += e;
      const float f = fmaf(y, e, sx);
      sx = e > 0.f ? f : sx;
      s_e[i + (i >> 5)] = e;
    }
    __syncthreads();
    const int a = max(v0, p * AT_THREADS) - p * AT_THREADS, b = min(v1, (p + PIECE) * AT_THREADS) - p * AT_THREADS;
    for (int i = a; i < b; ++i) run += s_e[i + (i >> 5)];
  }
  runs[(size_t)blockIdx.x * AT_THREADS + t] = run;
  z = wave_sum(z);                                         // fixed order: lanes by butterfly, waves ascending
  sx = wave_sum(sx);
  if ((t & 63) == 0) { sm[t >> 6] = z; sm2[t >> 6] = sx; }
  __syncthreads();
  if (t == 0) {
    z = sm[0]; sx = sm2[0];
    for (int w = 1; w < AT_WAVES; ++w) { z += sm[w]; sx += sm2[w]; }
    stats[blockIdx.x] = make_float4(m, z, logf(z) - sx / z, 0.f);
  }
}

__global__ __launch_bounds__(AT_THREADS) void k_accept_typical(const int32_t *parent, const int32_t *depth, int T, int K, int V,
                                                               const int32_t *tree_tok, const float *logits, const float4 *stats,
                                                               const float *runs, float inv_temp, float eps, float delta, const float *u,
                                                               int32_t *accept_len, int32_t *accept_path, int32_t *next_tok,
                                                               int32_t *best_node) {
  __shared__ float sm[AT_WAVES];
  __shared__ int s_pass[AMPH_MAX_TREE], s_parent[AMPH_MAX_TREE];
  __shared__ int s_key[AT_WAVES];
  __shared__ int s_best, s_run;
  __shared__ float s_exc;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const int32_t *tok = tree_tok + (size_t)b * T;
  const float ub = u[b];
  int dep = 0;
  if (t < T) {
    int pass = 1;                                          // the root
    const int j = parent[t], tk = tok[t];
    dep = depth[t];
    s_parent[t] = j;                                       // (the walks up the tree below would each be a chain of global loads)
    if (t > 0) {
      const size_t row = (size_t)b * T + j;
      const float4 st = stats[row];
      const bool known = tk >= 0 && tk < V;
      const float lt = logits[row * V + (known ? tk : 0)];
      const float p = expf((lt - st.x) * inv_temp) / st.y;
      pass = known && p > fminf(eps, delta * expf(-st.z));
    }
    s_pass[t] = pass;
  }
  if (t == 0) s_run = -1;
  __syncthreads();
  int key = -1;
  if (t < T) {
    bool ok = true;
    int j = t;
    for (int hop = 0; hop <= AMPH_MAX_HEADS_K && j > 0; ++hop) {
      if (!s_pass[j]) { ok = false; break; }
      j = s_parent[j];
    }
    if (ok) key = dep * 256 + (255 - t);
  }
  key = wave_max(key);
  if (lane == 0) s_key[t >> 6] = key;
  __syncthreads();
  int best_key = s_key[0];
  #pragma unroll
  for (int w = 1; w < (AMPH_MAX_TREE + WAVE - 1) / WAVE; ++w) best_key = max(best_key, s_key[w]);    // (the other waves hold no node)
  const int a = best_key >> 8, best = 255 - (best_key & 255);       // the root always qualifies
  // ---- the draw from p_best
  const size_t row = (size_t)b * T + best;
  const float *l = logits + row * V;
  const float4 st = stats[row];
  const float run = runs[row * AT_THREADS + t];
  if (t == 0) {
    accept_len[b] = a;
    best_node[b] = best;
    for (int dd = a + 1; dd <= K; ++dd) accept_path[(size_t)b * (K + 1) + dd] = -1;
    int j = best;
    for (int dd = a; dd >= 0 && j >= 0; --dd) { accept_path[(size_t)b * (K + 1) + dd] = j; j = s_parent[j]; }
  }
  const float target = ub * st.y;
  const int C = (V + AT_THREADS - 1) / AT_THREADS;
  // inclusive scan of the runs: inside a wave, then over the wave totals (ascending)
  float inc = run;
  #pragma unroll
  for (int off = 1; off < WAVE; off <<= 1) {
    const float o = __shfl_up(inc, off, WAVE);
    if (lane >= off) inc += o;
  }
  if (lane == 63) sm[t >> 6] = inc;
  __syncthreads();
  float base = 0.f;
  for (int w = 0; w < (t >> 6); ++w) base += sm[w];
  inc += base;
  const float prev = __shfl_up(inc, 1, WAVE);
  const float exc = lane ? prev : base;                   // exactly the thread before's inclusive sum
  // the sums never decrease with t and exc(t + 1) = inc(t): at most one thread sees the crossing inside its run
  if (exc <= target && inc > target) { s_run = t; s_exc = exc; }
  __syncthreads();
  const int r = s_run;
  if (r >= 0) {                                            // (uniform over the workgroup)
    if (t >= WAVE) return;
    // one wave walks the run: a token per lane, added up in order
    const int v0 = min(r * C, V), n = min(v0 + C, V) - v0;
    const float e = lane < n ? expf((l[min(v0 + lane, V - 1)] - st.x) * inv_temp) : 0.f;
    const unsigned long long live = __ballot(e > 0.f);
    float acc = s_exc;
    int pick = -1;
    for (int i = 0; i < n; ++i) {
      acc += __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(e), i));
      if (acc > target) { pick = v0 + i; break; }
    }
    if (pick < 0) pick = live ? v0 + 63 - __clzll(live) : v0;      // (acc and inc differ by rounding order only)
    if (t == 0) next_tok[b] = min(max(pick, 0), V - 1);
    return;
  }
  // no run crosses: the last token of non-zero probability
  int last_live = -1;
  for (int v = t; v < V; v += AT_THREADS)
    if (expf((l[v] - st.x) * inv_temp) > 0.f) last_live = v;
  last_live = wave_max(last_live);
  if (lane == 0) s_key[t >> 6] = last_live;
  __syncthreads();
  if (t == 0) {
    int pick = s_key[0];
    for (int w = 1; w < AT_WAVES; ++w) pick = max(pick, s_key[w]);
    next_tok[b] = min(max(pick, 0), V - 1);
  }
}

size_t accept_runs_floats(int rows) { return (size_t)rows * AT_THREADS; }

hipError_t launch_accept_typical(hipStream_t st, const int32_t *parent, const int32_t *depth, int T, int B, int K, int V,
                                 const int32_t *tree_tok, const float *logits, float temperature, float eps, float delta,
                                 const float *u, int32_t *accept_len, int32_t *accept_path, int32_t *next_tok,
                                 int32_t *best_node, float *stats_ws, float *runs_ws) {
  if (T < 1 || T > AMPH_MAX_TREE || V < 1 || !(temperature > 0.f)) return hipErrorInvalidValue;
  const float inv_temp = 1.0f / temperature;
  if (V > AT_MAX_RUN * AT_THREADS) return hipErrorInvalidValue;
  #define AT_STATS(N) hipLaunchKernelGGL((k_row_softmax_stats<N>), dim3(B * T), dim3(AT_THREADS), 0, st, logits, V, inv_temp, (float4 *)stats_ws, runs_ws)
  if (V <= 8 * AT_THREADS) AT_STATS(8); else if (V <= 32 * AT_THREADS) AT_STATS(32); else AT_STATS(64);
  #undef AT_STATS
  hipLaunchKernelGGL(k_accept_typical, dim3(B), dim3(AT_THREADS), 0, st, parent, depth, T, K, V, tree_tok, logits,
                     (const float4 *)stats_ws, (const float *)runs_ws, inv_temp, eps, delta, u, accept_len, accept_path, next_tok, best_node);
  return hipGetLastError();
}

// =====================================================================================================
// The loop around the step (Sec. 2 "Speculative Decoding"; Eq. 1 keeps one adaptation-layer cache row per
// committed position).
//   k_commit: for one (layer, batch element, head), the K/V rows of the accepted path's nodes 1..a move
//     from tree slots kv_len + node to kv_len + j (node 0, the root, already sits at kv_len).  All sources
//     are read before the first write (a destination may be another node's source).  In one more layer of the grid (the
//     first: its few workgroups have the longest way), row j <= a of h_new is the target's hidden state at path node j,
//     tok_new[j] the token that follows it (the next path node's token, or next_tok after the last), rows past a are zero,
//     and n_new = a + 1;
//   k_advance: kv_len += a + 1: a launch after the one above, whose workgroups have all read kv_len by then.
// A chain of latencies, so what can be asked for at once is: the lengths together with the whole path, then every accepted
// source.  Over deep caches it is bound by the values: lines of which two bytes move, read and written.  Measured (us by the
// kernel trace, k_commit; k_advance takes 1.3 behind it where the commits follow each other, up to 5 at the end of a long
// step), for 0, 1, 2, 3 and all nodes accepted in every sequence, against a version that read a source for every place of
// the path, accepted or not: 8 layers of 7B width, batch 4: 2.7 4.7 5.3 5.9 7.2 (4.3 5.9 6.3 6.7 7.9); 40 layers of 13B,
// batch 4: 4.9 19.3 20.2 22.1 29.0 (13.5 20.5 22.2 25.0 31.2); 60 layers of 33B, batch 4: 9.0 35.4 37.1 41.5 80.9
// (26.5 38.7 42.5 48.3 87.8).
// =====================================================================================================
template <int N> struct RowTag { static constexpr int value = N; };

template <typename T, int DH>
__global__ __launch_bounds__(256) void k_commit(T *k_caches, T *v_caches, int B, int n_heads, int max_kv, int T_nodes,
                                                const int32_t *kv_len, const int32_t *accept_len, const int32_t *accept_path, int K,
                                                int d, const float *hidden, const int32_t *tree_tok, const int32_t *next_tok,
                                                float *h_new, int32_t *tok_new, int32_t *n_new) {
  constexpr int PER = Elem<T>::PER;
  const int h = blockIdx.x, b = blockIdx.y, li = (int)blockIdx.z - (h_new ? 1 : 0), t = threadIdx.x;
  const int32_t *path = accept_path + (size_t)b * (K + 1);
  if (li < 0) {                                              // the draft's next rows
    const int a = min(max(accept_len[b], 0), K);
    for (int j = h; j <= K; j += n_heads) {
      const int node = min(max(path[j], 0), T_nodes - 1), node1 = min(max(path[min(j + 1, K)], 0), T_nodes - 1);
      float *dst = h_new + ((size_t)b * (K + 1) + j) * d;
      const float *src = hidden + ((size_t)b * T_nodes + node) * d;
      for (int k0 = t * 4; k0 < d; k0 += 4 * 1024) {         // four pieces are asked for before the first is stored
        float4 v[4];
        #pragma unroll
        for (int i = 0; i < 4; ++i)
          v[i] = j <= a ? *reinterpret_cast<const float4 *>(src + min(k0 + i * 1024, d - 4)) : make_float4(0.f, 0.f, 0.f, 0.f);
        #pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + i * 1024 < d) *reinterpret_cast<float4 *>(dst + k0 + i * 1024) = v[i];
      }
      if (t == 0) {
        tok_new[(size_t)b * (K + 1) + j] = j < a ? tree_tok[(size_t)b * T_nodes + node1] : j == a ? next_tok[b] : 0;
        if (j == 0) n_new[b] = a + 1;
      }
    }
    return;
  }
  // Thread t moves the 16-byte piece kp of key row kj, and of value rows vj, vj + VR, ... (the same for a whole wave) the dim ve
  // (a row's dims lie 64 bytes apart).
  constexpr int KPR = DH / PER, VR = 256 / DH, MAXI = AMPH_MAX_HEADS_K / VR;
  static_assert(AMPH_MAX_HEADS_K * KPR <= 256 && DH % WAVE == 0, "a thread for every piece of the keys; a wave for one value row");
  const int kj = 1 + t / KPR, kp = t % KPR, vj = 1 + __builtin_amdgcn_readfirstlane(t / DH), ve = t % DH;
  int L = kv_len[b], a = accept_len[b], kn = path[min(kj, K)], first = path[1];
  int vn[MAXI];
  #pragma unroll
  for (int i = 0; i < MAXI; ++i) vn[i] = path[min(vj + i * VR, K)];
  asm volatile("" : "+v"(L), "+v"(a), "+v"(kn), "+v"(first));         // one round trip: all are asked for ahead of the branches
  #pragma unroll
  for (int i = 0; i < MAXI; ++i) asm volatile("" : "+v"(vn[i]));
  L = __builtin_amdgcn_readfirstlane(L);
  a = min(__builtin_amdgcn_readfirstlane(a), K);
  if (L < 0 || L + T_nodes > max_kv || a < 1) return;       // the target pass wrote nothing (flagged there), or nothing moves
  const size_t head = (((size_t)li * B + b) * n_heads + h) * (size_t)max_kv * DH;
  T *kc = k_caches + head, *vc = v_caches + head;
  auto slot = [&](int node) { return L + min(max(node, 0), T_nodes - 1); };
  // Only what was accepted is read (a value row is DH lines): N value rows in this wave, in code without branches, as each
  // would have its loads wait for those before it.  Lanes without a key row re-read the first one's.
  auto move = [&](auto tag) {
    constexpr int N = decltype(tag)::value;
    const uint4 kr = ldg16(kc + k_tiled_index<T>(slot(kj <= a ? kn : first), kp * PER, DH));
    T vr[N > 0 ? N : 1];
    #pragma unroll
    for (int i = 0; i < N; ++i) vr[i] = vc[v_tiled_index<T>(slot(vn[i]), ve, DH)];
    __syncthreads();
    if (kj <= a) stg16(kc + k_tiled_index<T>(L + kj, kp * PER, DH), kr);
    #pragma unroll
    for (int i = 0; i < N; ++i) vc[v_tiled_index<T>(L + vj + i * VR, ve, DH)] = vr[i];
  };
  static_assert(MAXI == 2 || MAXI == 4, "the cases below");
  switch (a < vj ? 0 : (a - vj) / VR + 1) {
    case 0: move(RowTag<0>{}); break;
    case 1: move(RowTag<1>{}); break;
    case 2: move(RowTag<2>{}); break;
    case 3: move(RowTag<MAXI == 4 ? 3 : 2>{}); break;
    default: move(RowTag<MAXI>{}); break;
  }
}

__global__ __launch_bounds__(64) void k_advance(const int32_t *accept_len, int B, int K, int T_nodes, int max_kv, int32_t *kv_len) {
  const int b = threadIdx.x;                                // B <= 64
  if (b >= B) return;
  const int a = accept_len[b], L = kv_len[b];
  if (L >= 0 && L + T_nodes <= max_kv) kv_len[b] = L + min(max(a, 0), K) + 1;
}

template <typename T>
hipError_t launch_commit(hipStream_t st, void *k_caches, void *v_caches, int n_layers, int B, int n_heads, int d_h, int max_kv,
                         int T_nodes, int d, int K, int32_t *kv_len, const int32_t *accept_len, const int32_t *accept_path,
                         const int32_t *next_tok, const int32_t *tree_tok, const float *hidden, float *h_new, int32_t *tok_new,
                         int32_t *n_new) {
  if (K < 1 || K > AMPH_MAX_HEADS_K || (d_h != 64 && d_h != 128) || d % 4 || B > 64) return hipErrorInvalidValue;
  const int nz = n_layers + (h_new ? 1 : 0);
  #define COMMIT_LAUNCH(DH)                                                                                                      \
    hipLaunchKernelGGL((k_commit<T, DH>), dim3(n_heads, B, nz), dim3(256), 0, st, (T *)k_caches, (T *)v_caches, B, n_heads, max_kv, \
                       T_nodes, kv_len, accept_len, accept_path, K, d, hidden, tree_tok, next_tok, h_new, tok_new, n_new)
  if (nz > 0) { if (d_h == 128) COMMIT_LAUNCH(128); else COMMIT_LAUNCH(64); }
  #undef COMMIT_LAUNCH
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, st, accept_len, B, K, T_nodes, max_kv, kv_len);
  return hipGetLastError();
}
template hipError_t launch_commit<float>(hipStream_t, void *, void *, int, int, int, int, int, int, int, int, int32_t *,
                                         const int32_t *, const int32_t *, const int32_t *, const int32_t *, const float *,
                                         float *, int32_t *, int32_t *);
template hipError_t launch_commit<bf16_t>(hipStream_t, void *, void *, int, int, int, int, int, int, int, int, int32_t *,
                                          const int32_t *, const int32_t *, const int32_t *, const int32_t *, const float *,
                                          float *, int32_t *, int32_t *);

// =====================================================================================================
// Row-major [max_kv, d_h] caches <-> the step-tiled storage of the verification attention (formulas: header of
// the C ABI, k_tiled_index / v_tiled_index).  Pure data movement, bound by HBM: a wave moves one key step of one cache
// (keys or values; 32 rows in bf16, 16 in float: DH / 16 pieces of 16 bytes per lane, all requested before the first is
// used), so both sides of the copy are one contiguous block of 4 or 8 KB and every line of it is touched by one wave.
//   keys    lane pieces go straight across: 4 adjacent rows of a 64-byte column are 256 contiguous bytes of the tile;
//   values  a lane holds DH / 16 adjacent rows of PER adjacent dims and turns them round in registers: a dim's rows
//           are adjacent in the tile.
// (One element at a time the values' side was 2-byte accesses 64 bytes apart: 2.3 GB of pack and unpack over 32 layers
// of 7B caches 1440 us, 1.6 TB/s; this way 395 us, 5.8 TB/s.)
// The launch asks for LDS that it does not use, so that three workgroups (six of half the bytes at 64-wide heads) share a
// compute unit: as many as the registers allow have too many streams open (us, pack / unpack of the 7B caches, workgroups a
// unit: 8 211 / 214, 7 210 / 208, 5 204 / 206, 4 200 / 202, 3 196 / 198; smaller conversions the same).
// =====================================================================================================
constexpr int kvl_lds_bytes(int d_h) { return d_h == 128 ? 52 * 1024 : 26 * 1024; }

template <typename T, int DH, bool TO_TILED>
__global__ __launch_bounds__(256) void k_kv_layout(const T *k_src, const T *v_src, T *k_dst, T *v_dst, int n_caches, int max_kv) {
  constexpr int PER = Elem<T>::PER, KSTEP = 4 * PER, UN = DH / 16, LPR = DH / PER;   // LPR lanes cover a row
  constexpr int STEP_ELEMS = KSTEP * DH;
  typedef T frag __attribute__((ext_vector_type(PER)));
  typedef T run __attribute__((ext_vector_type(UN)));      // the rows of one dim that a lane holds
  const int lane = threadIdx.x & 63, steps = max_kv / KSTEP;
  const int li = lane % LPR, grp = lane / LPR;
  const int kinds = (k_src && v_src) ? 2 : 1;
  const long long units = (long long)n_caches * steps * kinds;
  for (long long u = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); u < units; u += (long long)gridDim.x * 4) {
    const bool keys = kinds == 2 ? (u & 1) == 0 : k_src != nullptr;
    const size_t base = (size_t)(kinds == 2 ? u >> 1 : u) * STEP_ELEMS;     // a step is contiguous on both sides
    frag x[UN];
    if (keys) {
      // piece j of a lane: row j * (64 / LPR) + grp, dims li * PER ..
      #pragma unroll
      for (int j = 0; j < UN; ++j) {
        const int row = j * (64 / LPR) + grp;
        const size_t o = TO_TILED ? (size_t)row * DH + li * PER : k_tiled_index<T>(row, li * PER, DH);
        x[j] = __builtin_nontemporal_load(reinterpret_cast<const frag *>(k_src + base + o));
      }
      #pragma unroll
      for (int j = 0; j < UN; ++j) {
        const int row = j * (64 / LPR) + grp;
        const size_t o = TO_TILED ? k_tiled_index<T>(row, li * PER, DH) : (size_t)row * DH + li * PER;
        *reinterpret_cast<frag *>(k_dst + base + o) = x[j];
      }
    } else {
      // rows grp * UN + j, j < UN
      run y[PER];
      if (TO_TILED) {
        #pragma unroll
        for (int j = 0; j < UN; ++j)
          x[j] = __builtin_nontemporal_load(reinterpret_cast<const frag *>(v_src + base + (size_t)(grp * UN + j) * DH + li * PER));
        #pragma unroll
        for (int e = 0; e < PER; ++e) {
          #pragma unroll
          for (int j = 0; j < UN; ++j) y[e][j] = x[j][e];
          *reinterpret_cast<run *>(v_dst + base + v_tiled_index<T>(grp * UN, li * PER + e, DH)) = y[e];
        }
      } else {
        #pragma unroll
        for (int e = 0; e < PER; ++e)
          y[e] = __builtin_nontemporal_load(reinterpret_cast<const run *>(v_src + base + v_tiled_index<T>(grp * UN, li * PER + e, DH)));
        #pragma unroll
        for (int j = 0; j < UN; ++j) {
          #pragma unroll
          for (int e = 0; e < PER; ++e) x[j][e] = y[e][j];
          *reinterpret_cast<frag *>(v_dst + base + (size_t)(grp * UN + j) * DH + li * PER) = x[j];
        }
      }
    }
  }
}

template <typename T>
hipError_t launch_kv_layout(hipStream_t st, const void *k_src, const void *v_src, void *k_dst, void *v_dst, int n_caches,
                            int max_kv, int d_h, bool to_tiled) {
  if (n_caches < 1 || n_caches > 65535 * 16 || max_kv % 32 || (d_h != 64 && d_h != 128)) return hipErrorInvalidValue;
  const long long units = (long long)n_caches * (max_kv / (4 * Elem<T>::PER)) * ((k_src && v_src) ? 2 : 1);
  const dim3 grid((unsigned)std::min<long long>((units + 3) / 4, 16384)), block(256);
  #define KVL(DH_, W_) hipLaunchKernelGGL((k_kv_layout<T, DH_, W_>), grid, block, kvl_lds_bytes(DH_), st, (const T *)k_src, (const T *)v_src, \
                                          (T *)k_dst, (T *)v_dst, n_caches, max_kv)
  if (d_h == 64) { if (to_tiled) KVL(64, true); else KVL(64, false); }
  else { if (to_tiled) KVL(128, true); else KVL(128, false); }
  #undef KVL
  return hipGetLastError();
}
template hipError_t launch_kv_layout<float>(hipStream_t, const void *, const void *, void *, void *, int, int, int, bool);
template hipError_t launch_kv_layout<bf16_t>(hipStream_t, const void *, const void *, void *, void *, int, int, int, bool);

// =====================================================================================================
// Row-wise RMSNorm for the target path, fused with the fold of the previous GEMM's partial slabs:
//   x[m] (+)= sum_s slabs[s][m]   (or x[m] = embed[tok[m]] on entry to the first layer)
//   xn[m] = x[m] / rms(x[m]) * g  stored as T for the matrix cores; hidden_out optionally in float32.
// One 1024-thread workgroup per row, one 16-byte piece of every operand per thread and pass.  The
// number of slabs, the source of the row and the number of passes are template parameters so that the
// body is straight-line code: every load of a pass is issued before the first use (a run-time loop over
// slabs costs one memory round trip per slab).  d <= 8192.
// =====================================================================================================
template <typename T, int S, bool EMB, int NP>
__global__ __launch_bounds__(1024) void k_norm_fold(float *x, const T *embed, const int32_t *tok, int vocab,
                                                    const float *slabs, size_t slab_stride, const T *g, int d,
                                                    float eps, T *xn, float *hidden_out, uint32_t *dev_status, int xn_tiles,
                                                    RopeTable rope, int rows) {
  __shared__ float red[16];
  const int tid = threadIdx.x;
  // A KB of the tiled activations holds 16 rows: they are dealt to one XCD (workgroups 8 apart), so that its L2 sees whole lines.
  // With neighbouring rows on neighbouring XCDs every line left eight L2s in pieces (target pass, us: 33B over 384 rows 654 / 648, 7B
  // over 512 617 / 612, 13B over 128 270.7 / 268.3).
  const int j = blockIdx.x >> 3, row = xn_tiles ? ((j >> 4) * 8 + (blockIdx.x & 7)) * 16 + (j & 15) : blockIdx.x;
  if (row >= rows) return;                                         // (whole workgroup)
  float *xr = x + (size_t)row * d;
  int t = 0;
  if (EMB) {
    t = tok[row];
    if (t < 0 || t >= vocab) { if (tid == 0) atomicOr(dev_status, 4u); t = 0; }
  }
  float v[NP][4], gk[NP][4], p[NP][S > 0 ? S : 1][4];
  #pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int k = (tid + i * 1024) * 4, kk = k < d ? k : 0;      // pieces past the row re-read its start, unused
    if (EMB) load4<T>(embed + (size_t)t * d + kk, v[i]);
    else load4<float>(xr + kk, v[i]);
    #pragma unroll
    for (int s = 0; s < S; ++s) load4<float>(slabs + (size_t)s * slab_stride + (size_t)row * d + kk, p[i][s]);
    load4<T>(g + kk, gk[i]);
  }
  if (EMB && rope.cs) {
    // the pass's RoPE table rides on the kernel that starts the pass (one launch fewer): row `row` of
    // (cos, sin) of pos * theta^(-2e/d_h), e < d_h/2, the same for every layer
    const int half = rope.d_h / 2;
    for (int e = tid; e < half; e += 1024) {
      const float inv_freq = exp2f(-2.0f * (float)e / (float)rope.d_h * log2f(rope.theta));
      float sn, c;
      sincosf((float)rope.pos[row] * inv_freq, &sn, &c);
      rope.cs[(size_t)row * half + e] = make_float2(c, sn);
    }
  }
  float ss = 0.f;
  #pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int k = (tid + i * 1024) * 4;
    #pragma unroll
    for (int s = 0; s < S; ++s) {
      #pragma unroll
      for (int j = 0; j < 4; ++j) v[i][j] += p[i][s][j];
    }
    if (k < d) {
      if (EMB || S > 0) store4<float>(xr + k, v[i]);
      #pragma unroll
      for (int j = 0; j < 4; ++j) ss = fmaf(v[i][j], v[i][j], ss);
    }
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  #pragma unroll
  for (int w = 0; w < 16; ++w) tot += red[w];
  const float rs = rsqrtf(tot / (float)d + eps);
  #pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int k = (tid + i * 1024) * 4;
    if (k < d) {
      float o[4];
      #pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = v[i][j] * rs * gk[i][j];
      store4<T>(xn_tiles ? xn + xt_index<T>(row, k, xn_tiles) : xn + (size_t)row * d + k, o);
      if (hidden_out) store4<float>(hidden_out + (size_t)row * d + k, o);
    }
  }
}

template <typename T>
hipError_t launch_norm_fold(hipStream_t st, float *x, const void *embed, const int32_t *tok, int vocab,
                            const float *slabs, int S, size_t slab_stride, const void *g, int rows, int d, float eps,
                            void *xn, float *hidden_out, uint32_t *dev_status, int xn_tiles, RopeTable rope) {
  if (d % 4 || d > 8192) return hipErrorInvalidValue;
  if (tok && S != 0) return hipErrorInvalidValue;                  // the embedding gather starts a fresh residual stream
  if (rope.cs && (!tok || !rope.pos || rope.d_h < 2)) return hipErrorInvalidValue;   // the table is written by the embedding instance
  const int np = d > 4096 ? 2 : 1, wgs = xn_tiles ? (rows + 127) / 128 * 128 : rows;
  #define NF_LAUNCH(S_, EMB_, NP_)                                                                                  \
    hipLaunchKernelGGL((k_norm_fold<T, S_, EMB_, NP_>), dim3(wgs), dim3(1024), 0, st, x, (const T *)embed, tok,     \
                       vocab, slabs, slab_stride, (const T *)g, d, eps, (T *)xn, hidden_out, dev_status, xn_tiles, rope, rows)
  #define NF_CASE(S_)                                                                                               \
    case S_: if (np == 1) NF_LAUNCH(S_, false, 1); else NF_LAUNCH(S_, false, 2); break
  if (tok) {
    if (np == 1) NF_LAUNCH(0, true, 1); else NF_LAUNCH(0, true, 2);
  } else {
    switch (S) {
      NF_CASE(0); NF_CASE(1); NF_CASE(2); NF_CASE(4); NF_CASE(8);
      default: return hipErrorInvalidValue;
    }
  }
  #undef NF_CASE
  #undef NF_LAUNCH
  return hipGetLastError();
}
template hipError_t launch_norm_fold<float>(hipStream_t, float *, const void *, const int32_t *, int, const float *, int,
                                            size_t, const void *, int, int, float, void *, float *, uint32_t *, int, RopeTable);
template hipError_t launch_norm_fold<bf16_t>(hipStream_t, float *, const void *, const int32_t *, int, const float *, int,
                                             size_t, const void *, int, int, float, void *, float *, uint32_t *, int, RopeTable);

}  // namespace amph

// Matrix-core form of the draft path's projections (Sec. 3.1 Eq. 1, Sec. 3.2 Eq. 2-6): float32 activation rows
// against row-major bf16 weights, for the row counts at which the vector kernels of gemv.hip stop being bound by HBM
// (catch-up rows of the loop, batches).  One pass over the weights serves up to 48 rows.
//
// Precision.  The activations are float32 and stay so: an element x is cut into three bf16 pieces by truncation,
// x = hi + mid + lo, which is exact (24 = 8 + 8 + 8 significant bits), and every weight fragment is multiplied with
// all three; products of two bf16 values are exact in the float32 accumulator.
//
// The matrix cores' accumulator rounds down (measured: a bias of -3.5e-6 over 17920 positive terms when one
// accumulator runs through the whole axis), so each step's three products start from zero and are added to the running
// sum by the vector ALU, which rounds to nearest; and every other wave multiplies the negated weights, so that what is
// left of the bias cancels in the sum over the waves.
//
// Weights are finite (as gemv.hip takes them to be: its padding multiplies them by zero too); an infinite or NaN activation
// gives what it gives there.
//
// Shape.  A workgroup owns NB row blocks of 16 weight rows, all activation rows (NT tiles of 16) and the whole reduction axis,
// or one of up to DRAFT_MM_SPLITS parts of it (dm_pick), whose sums k_draft_fold adds up.  Its waves have two roles:
//   * 2 loader waves stream the weight rows from HBM and the activation rows from L2 into a ring of LDS stages
//     (global-to-LDS loads).  A matrix-core operand fragment is 16 rows x 64 bytes; fetched from row-major rows directly
//     it is 16 half cache lines per load, which a CU's vector L1 serves at a quarter of the rate of whole lines.  So a
//     load takes a few hundred contiguous bytes of each of its rows, and the 16-byte pieces of a row are permuted on the
//     way in (piece p of row r at slot p ^ (r % 16)) so that the fragment reads from LDS are free of bank conflicts.
//     The activations travel in the same ring because a CU's loads return in order: fetched into registers by the math
//     waves they queue behind the ring's worth of weights in flight (7B W_down over 5 rows: 53 us).
//   * KW math waves split the reduction axis: wave w takes step w (64 bytes of a weight row) of every stage (and step w + KW
//     of a stage of 1024 bytes), against all NB blocks and NT tiles, so each activation element is read from LDS and cut into its pieces once per workgroup.  A
//     step costs about 45 vector instructions per tile whatever NB is, which what a compute unit takes in mostly hides: twice the
//     math waves, sharing the tiles, changed nothing (nor did reading the next step's operands ahead of this one's arithmetic).
// The KW partial sums meet in LDS after the loop and are added in a fixed order; RMSNorm's 1/rms of a row is
// applied there too (the waves collect the squares of the elements they saw).
#include "kernels.h"
#include <algorithm>

namespace amph {

constexpr int DM_NL = 2;                        // loader waves
constexpr int DM_MAX_R = 14;                    // stages in the ring, at most

enum DmEpi { DM_LINEAR = 0, DM_FC = 1, DM_SALQKV = 2, DM_SWIGLU = 3, DM_HEADMLP = 4, DM_LMTOPK = 5 };

struct DmArgs {
  const bf16_t *w0, *w1, *w2;     // stacked matrices of seg_rows rows of Kd elements each
  int n_seg, seg_rows, Kd, M;
  const float *x;                 // [M, ldx] float32 (DM_FC: u; DM_HEADMLP: h1)
  int ldx;
  const bf16_t *gain;             // RMSNorm weights (DM_SALQKV, DM_SWIGLU)
  float eps;
  float *o0, *o1, *o2;            // outputs [M, ldo] per segment
  int ldo;
  const float *res;               // DM_LINEAR: residual [M, ldo] or NULL
  LastRows last;                  // DM_LINEAR, DM_FC with one matrix
  // DM_FC
  const bf16_t *embed; const int32_t *tok; int vocab;
  // DM_SALQKV
  int n_heads, d_h, max_kv, row0, R;
  float theta;
  const int32_t *sal_len, *n_valid;
  bf16_t *kv_stage;
  // DM_HEADMLP
  const float *x2; const bf16_t *pe; int K;
  // DM_LMTOPK
  float *logits, *cand_v; int *cand_i; int topk;
  uint32_t *dev_status;
  float *slabs;                   // DM_LINEAR, DM_FC with split axis: [S][M][seg_rows] partial sums, or NULL: the axis stays whole
  int blocks, ring, stage_bytes;  // row blocks of the launch; stages in the LDS ring and their bytes
};

template <int NB, int NT, int CB_> struct DmStage {
  static constexpr int CB = CB_;                                     // bytes of one weight row per stage
  static constexpr int KW = CB == 256 ? 4 : 8;                       // math waves
  static constexpr int SPW = CB / 64 / KW;                           // steps of each per stage
  static constexpr int THREADS = 64 * (KW + DM_NL);
  static constexpr int WB = NB * 16 * CB;                            // bytes of weights per stage
  static constexpr int RPI = 1024 / CB;                              // weight rows per load instruction
  static constexpr int LPW = NB * 16 / RPI / DM_NL;                  // weight loads per loader wave and stage
  static constexpr int XRB = 2 * CB;                                 // bytes of one float32 activation row per stage
  static constexpr int LPX = XRB > 1024 ? XRB / 1024 : 1;            // load instructions per activation row ...
  static constexpr int RPX = XRB > 1024 ? 1 : 1024 / XRB;            // ... or rows per instruction
};
// A wave of a launch with few row blocks adds its steps up in runs of DM_RUN (shorter chains of roundings): its reduction
// axis may be long (W_down; error over 17920 terms 2.2e-7 -> 1.1e-7, the vector kernels' 1.7e-7).  With more blocks the
// second set of sums would cost the registers that let two workgroups share a compute unit, and the axis is the model
// width (error 1.4e-7 over 6656 terms without runs, the vector kernels' 1.9e-7).
constexpr int DM_RUN = 16, DM_RUNS_NB = 2, DM_LONG = 8192;
constexpr int DM_GAIN_B = 1024;                 // RMSNorm weights of a stage

template <int N> struct DmTag { static constexpr int value = N; };

template <int N> __device__ __forceinline__ void dm_wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}
// waits until at most n (wave-uniform, below 64) of this wave's vector-memory operations are outstanding
template <int LO = 0, int HI = 64> __device__ __forceinline__ void dm_wait_at_most(int n) {
  if constexpr (HI - LO == 1) {
    dm_wait_vm<LO>();
  } else {
    constexpr int MID = (LO + HI) / 2;
    if (n < MID) dm_wait_at_most<LO, MID>(n); else dm_wait_at_most<MID, HI>(n);
  }
}

// the upper halves of two floats as two adjacent bf16 (truncation)
__device__ __forceinline__ unsigned dm_hi2(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}

// x = hi + mid + lo for 8 floats, each piece a bf16 fragment.  With weights (NORM) x is f * w, of which what lies below hi is taken
// from the unrounded product.  Infinities would leave NaN in the lower pieces (inf - inf): INF puts them in hi alone.
template <bool NORM, bool INF> __device__ __forceinline__ void dm_split(const float (&x)[8], const float (&f)[8], const float (&w)[8], uint4 &hi, uint4 &mid, uint4 &lo) {
  float r[8], q[8];
  #pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float top = __uint_as_float(__float_as_uint(x[i]) & 0xffff0000u);
    r[i] = NORM ? fmaf(f[i], w[i], -top) : x[i] - top;
    q[i] = r[i] - __uint_as_float(__float_as_uint(r[i]) & 0xffff0000u);
    if (INF && __builtin_amdgcn_classf(x[i], 0x204)) { r[i] = 0.f; q[i] = 0.f; }           // +-infinity
  }
  hi = make_uint4(dm_hi2(x[0], x[1]), dm_hi2(x[2], x[3]), dm_hi2(x[4], x[5]), dm_hi2(x[6], x[7]));
  mid = make_uint4(dm_hi2(r[0], r[1]), dm_hi2(r[2], r[3]), dm_hi2(r[4], r[5]), dm_hi2(r[6], r[7]));
  lo = make_uint4(dm_hi2(q[0], q[1]), dm_hi2(q[2], q[3]), dm_hi2(q[4], q[5]), dm_hi2(q[6], q[7]));
}

// 16 bytes a lane from base + off + at (off a lane's own, at the wave's) to LDS, lane by lane.  Nothing is written for a lane past `bytes`.
template <int AUX> __device__ __forceinline__ void dm_load_lds(const void *base, unsigned bytes, unsigned char *lds, int off, int at) {
#ifdef __HIP_DEVICE_COMPILE__                              // (the host's pass refuses 16 bytes)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000),
                                           (__attribute__((address_space(3))) void *)lds, 16, off, at, 0, AUX);
#endif
}

// Weight rows r16, r16 + 1, .. of block blk that lie next to each other (up to a multiple of eight): their matrix, the first one's row
// in it.  Rows past the end re-read the last row; they are never stored.  q and k blocks: 8 rows of a head and their 8 RoPE partners;
// gate/up blocks: 8 rows of each matrix.
struct DmRows { const bf16_t *w; int n, rows; };
template <int EPI>
__device__ __forceinline__ DmRows dm_rows(const DmArgs &a, int blk, int r16) {
  if (EPI == DM_SWIGLU) return {r16 >= 8 ? a.w1 : a.w0, min(blk * 8 + (r16 & 7), a.seg_rows - 1), a.seg_rows};
  const int bps = (a.seg_rows + 15) >> 4;
  if (EPI == DM_HEADMLP) {                                 // (one head a workgroup)
    const int seg = blockIdx.y;
    return {a.w0 + (size_t)seg * a.seg_rows * a.Kd, min((blk - seg * bps) * 16 + r16, a.seg_rows - 1), a.seg_rows};
  }
  const int seg = a.n_seg == 1 ? 0 : (blk >= 2 * bps ? 2 : blk >= bps ? 1 : 0), bl = blk - seg * bps;
  int n = bl * 16 + r16;
  if (EPI == DM_SALQKV && seg < 2) {
    const int bph = a.d_h >> 4;
    n = (bl / bph) * a.d_h + (bl % bph) * 8 + (r16 & 7) + ((r16 >= 8) ? a.d_h / 2 : 0);
  }
  return {seg == 0 ? a.w0 : seg == 1 ? a.w1 : a.w2, min(n, a.seg_rows - 1), a.seg_rows};
}

template <int EPI, int NB, int NT, int CB_>
__global__ __launch_bounds__((DmStage<NB, NT, CB_>::THREADS)) void k_draft_mm(const DmArgs a) {
  using C = DmStage<NB, NT, CB_>;
  constexpr int CB = C::CB, KW = C::KW, SPW = C::SPW, THREADS = C::THREADS, LPW = C::LPW, RPI = C::RPI, XRB = C::XRB, RPX = C::RPX;
  constexpr bool NORM = EPI == DM_SALQKV || EPI == DM_SWIGLU;
  constexpr bool RUNS = NB <= DM_RUNS_NB;
  extern __shared__ __align__(16) unsigned char dm_lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  // DM_HEADMLP: a workgroup's blocks belong to one head (its rows read one of two sources)
  const int bps = (a.seg_rows + 15) >> 4;
  const int head = EPI == DM_HEADMLP ? blockIdx.y : 0;
  const int b0 = blockIdx.x * NB;                          // first block (of the head)
  const int bl_last = (EPI == DM_HEADMLP ? bps : a.blocks) - 1;
  const int Kb = a.Kd * 2;
  const int P_all = (Kb + CB - 1) / CB;                    // stages of the whole axis; this workgroup's are [Pa, P)
  const int S = gridDim.z, Pa = (int)((unsigned)(P_all * blockIdx.z) / (unsigned)S), P = (int)((unsigned)(P_all * (blockIdx.z + 1)) / (unsigned)S);
  const int Kx = EPI == DM_FC ? a.Kd / 2 : a.Kd;           // float32 columns
  const int Pu = EPI == DM_FC ? P_all / 2 : P_all;         // stages whose activations are float32 (DM_FC: then the embeddings, bf16)
  const int R = a.ring, SB = a.stage_bytes;
  auto blk_of = [&](int b) { return head * bps + min(b0 + b, bl_last); };
  const float *xbase = (EPI == DM_HEADMLP && head >= a.K / 2) ? a.x2 : a.x;

  f32x4 acc[NB][NT], sum[RUNS ? NB : 1][RUNS ? NT : 1];    // long axes: acc holds runs of DM_RUN steps, sum the runs' total
  #pragma unroll
  for (int b = 0; b < NB; ++b)
    #pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[b][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (RUNS) sum[b][t] = acc[b][t];
    }
  float ss[NT];
  #pragma unroll
  for (int t = 0; t < NT; ++t) ss[t] = 0.f;

  if (wave >= KW) {
    // ------------------------------------------------------------------------------- loader wave
    // Loader l takes weight loads l * LPW .. and every other activation load; loader 1 also the RMSNorm weights.
    // Its loads go through buffer descriptors: what a lane adds to a load's base stays the same through the launch, and the stage
    // is a scalar offset.  Pieces past a row's end read what follows, past the end of the matrix nothing: what LDS holds there is not
    // looked at.  (With a dozen vector instructions of addresses for every load, on a SIMD that a math wave keeps busy, issuing the
    // 32 loads of a stage of 40 rows set the pace.  us, so / now: 40 rows QKV 12288 x 4096 44 / 39, W_down 4096 x 11008 32 / 27; 32 rows
    // 12288 x 4096 36 / 28, the LM head 32000 x 4096 75 / 71; 24 rows 35840 x 6656 111 / 102; five rows the same.)
    const int l = wave - KW;
    constexpr int PPR = CB / 16, PPX = XRB / 16;           // 16-byte pieces of a weight / float32 activation row per stage
    const unsigned char *wbase[LPW];
    unsigned wbytes[LPW];
    int wo[LPW];
    #pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const int r0 = (l * LPW + j) * RPI;                  // first row of the load in the stage: block r0 / 16, row r0 % 16 of it
      const DmRows rw = dm_rows<EPI>(a, blk_of(r0 >> 4), r0 & 15);
      const size_t left = (size_t)(rw.rows - rw.n) * Kb;
      wbase[j] = (const unsigned char *)rw.w + (size_t)rw.n * Kb;
      wbytes[j] = left < 0xffffffffu ? (unsigned)left : 0xffffffffu;
      wo[j] = min(lane / PPR, rw.rows - 1 - rw.n) * Kb + ((lane % PPR) ^ ((r0 + lane / PPR) & 15)) * 16;   // the piece that belongs at this lane's slot
    }
    const int nx = (a.M + RPX - 1) / RPX * C::LPX, ne = EPI == DM_FC ? (a.M + RPI - 1) / RPI : 0;     // activation loads per stage
    constexpr int XMAX = (NT * 16 / RPX * C::LPX + 1) / 2, EMAX = EPI == DM_FC ? (NT * 16 / RPI + 1) / 2 : 1;
    const unsigned xbytes = (unsigned)(((a.M - 1) * a.ldx + Kx) * 4);
    int xo[XMAX];
    #pragma unroll
    for (int j = 0; j < XMAX; ++j) {                       // rows past the end re-read the last one; never stored
      const int i = l + 2 * j, row = C::LPX > 1 ? i / C::LPX : i * RPX + lane / PPX, pl = C::LPX > 1 ? (i % C::LPX) * 64 + lane : lane % PPX;
      xo[j] = min(row, a.M - 1) * a.ldx * 4 + (pl ^ (row & 15)) * 16;
    }
    const unsigned char *esrc[EMAX];                       // DM_FC: embedding rows of this lane's loads
    if (EPI == DM_FC) {
      #pragma unroll
      for (int j = 0; j < EMAX; ++j) {
        const int row = (l + 2 * j) * RPI + lane / PPR, tk = a.tok[min(row, a.M - 1)];
        esrc[j] = (const unsigned char *)(a.embed + (size_t)((tk < 0 || tk >= a.vocab) ? 0 : tk) * a.ldx) + ((lane % PPR) ^ (row & 15)) * 16;
      }
    }
    const int go = min(lane % PPR, 63) * 16;
    const int cu = LPW + (nx - l + 1) / 2 + ((NORM && l == 1) ? 1 : 0), ce = LPW + (ne - l + 1) / 2;   // loads per stage
    typedef __attribute__((address_space(3))) void Lds;
    auto issue = [&](int p, int slot) {
      unsigned char *lp = dm_lds + (size_t)slot * SB;
      #pragma unroll
      for (int j = 0; j < LPW; ++j)
        dm_load_lds<2>(wbase[j], wbytes[j], lp + (l * LPW + j) * 1024, wo[j], p * CB);   // non-temporal
      unsigned char *xp = lp + C::WB;
      if (EPI == DM_FC && p >= Pu) {
        #pragma unroll
        for (int j = 0; j < EMAX; ++j)
          if (l + 2 * j < ne)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(esrc[j] + (p - Pu) * CB),
                                             (Lds *)(xp + (l + 2 * j) * 1024), 16, 0, 0);
      } else {
        #pragma unroll
        for (int j = 0; j < XMAX; ++j)
          if (l + 2 * j < nx) dm_load_lds<0>(xbase, xbytes, xp + (l + 2 * j) * 1024, xo[j], p * XRB);
        if (NORM && l == 1) dm_load_lds<0>(a.gain, Kb, lp + SB - DM_GAIN_B, go, p * CB);
      }
    };
    const int pro = P - Pa < R - 1 ? P - Pa : R - 1;
    for (int p = 0; p < pro; ++p) issue(Pa + p, p);
    int fill = pro;                                        // slot of the next stage to request
    for (int p = Pa; p < P; ++p) {
      const int newest = (p + R - 2 < P - 1) ? p + R - 2 : P - 1;
      const int nu = max(min(newest, Pu - 1) - p, 0), nn = newest - p;     // stages requested after p: float32 ones, all
      dm_wait_at_most(nu * cu + (nn - nu) * ce);           // stage p has landed
      asm volatile("s_barrier" ::: "memory");              // math waves may read stage p; they are done with stage p - 1
      if (p + R - 1 < P) {
        issue(p + R - 1, fill);
        if (++fill == R) fill = 0;
      }
    }
  } else {
    // --------------------------------------------------------------------------------- math wave
    bool elive[NT];                                        // DM_FC: whether the token is in range (otherwise its embedding is zero)
    if (EPI == DM_FC) {
      #pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int m = t * 16 + r16, tk = a.tok[min(m, a.M - 1)];
        elive[t] = tk >= 0 && tk < a.vocab;
        if (!elive[t] && m < a.M && blockIdx.x == 0 && g == 0 && wave == 0) atomicOr(a.dev_status, 4u);
      }
    }
    const unsigned sgn = (wave & 1) ? 0x80008000u : 0u;
    int slot = 0;
    for (int p = Pa; p < P; ++p) {
      // A bare barrier; the LDS reads of the stage before are waited for first, since its slot is refilled behind it.
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const unsigned char *sb = dm_lds + slot * SB, *sx = sb + C::WB;
      if (++slot == R) slot = 0;
      #pragma unroll
      for (int j = 0; j < SPW; ++j) {
        const int s = j * KW + wave, k = p * (CB / 2) + s * 32;          // step of the stage; its first column
        uint4 wf[NB];
        #pragma unroll
        for (int b = 0; b < NB; ++b) wf[b] = *reinterpret_cast<const uint4 *>(sb + (b * 16 + r16) * CB + (((s * 4 + g) ^ r16) * 16));
        if (EPI == DM_FC && p >= Pu) {                       // an embedding row is bf16 already
          #pragma unroll
          for (int t = 0; t < NT; ++t) {
            uint4 e = *reinterpret_cast<const uint4 *>(sx + (t * 16 + r16) * CB + (((s * 4 + g) ^ r16) * 16));
            if (!elive[t]) e = make_uint4(0u, 0u, 0u, 0u);
            e.x ^= sgn; e.y ^= sgn; e.z ^= sgn; e.w ^= sgn;
            #pragma unroll
            for (int b = 0; b < NB; ++b) acc[b][t] += mma16<bf16_t>(wf[b], e, (f32x4){0.f, 0.f, 0.f, 0.f});
          }
        } else {
          float gk[8];
          if (NORM) Elem<bf16_t>::unpack(*reinterpret_cast<const uint4 *>(sb + SB - DM_GAIN_B + (s * 4 + g) * 16), gk);
          if (NB <= 2 * NT) {                                // the sign goes where it takes fewer instructions
            #pragma unroll
            for (int b = 0; b < NB; ++b) { wf[b].x ^= sgn; wf[b].y ^= sgn; wf[b].z ^= sgn; wf[b].w ^= sgn; }
          }
          float f[NT][8], x[NT][8], top = 0.f;               // top: the largest magnitude (NaN aside)
          #pragma unroll
          for (int t = 0; t < NT; ++t) {
            const unsigned char *xr = sx + (t * 16 + r16) * XRB;
            float (&ft)[8] = f[t];
            float lo4[4], hi4[4];
            Elem<float>::unpack(*reinterpret_cast<const uint4 *>(xr + (((s * 8 + g * 2) ^ r16) * 16)), lo4);
            Elem<float>::unpack(*reinterpret_cast<const uint4 *>(xr + (((s * 8 + g * 2 + 1) ^ r16) * 16)), hi4);
            #pragma unroll
            for (int e = 0; e < 4; ++e) { ft[e] = lo4[e]; ft[4 + e] = hi4[e]; }
          }
          const bool ends = k + 32 > a.Kd;                   // (uniform) the reduction axis ends in this step
          if (ends && k + g * 8 >= a.Kd) {                   // (what lies there in LDS is anything)
            #pragma unroll
            for (int b = 0; b < NB; ++b) wf[b] = make_uint4(0u, 0u, 0u, 0u);
            #pragma unroll
            for (int e = 0; e < 8; ++e) gk[e] = 0.f;
            #pragma unroll
            for (int t = 0; t < NT; ++t)
              #pragma unroll
              for (int e = 0; e < 8; ++e) f[t][e] = 0.f;      // (Kd is a multiple of 8)
          }
          #pragma unroll
          for (int t = 0; t < NT; ++t) {
            if (NORM) {
              #pragma unroll
              for (int e = 0; e < 8; ++e) ss[t] = fmaf(f[t][e], f[t][e], ss[t]);
            }
            if (NB > 2 * NT) {
              #pragma unroll
              for (int e = 0; e < 8; ++e) f[t][e] = __uint_as_float(__float_as_uint(f[t][e]) ^ (sgn & 0x80000000u));
            }
            #pragma unroll
            for (int e = 0; e < 8; ++e) { x[t][e] = NORM ? f[t][e] * gk[e] : f[t][e]; top = fmaxf(top, fabsf(x[t][e])); }
          }
          auto multiply = [&](auto tag) {
            #pragma unroll
            for (int t = 0; t < NT; ++t) {
              uint4 hi, mid, lo;
              dm_split<NORM, decltype(tag)::value != 0>(x[t], f[t], gk, hi, mid, lo);
              f32x4 d[NB];
              #pragma unroll
              for (int b = 0; b < NB; ++b) d[b] = mma16<bf16_t>(wf[b], lo, (f32x4){0.f, 0.f, 0.f, 0.f});
              #pragma unroll
              for (int b = 0; b < NB; ++b) d[b] = mma16<bf16_t>(wf[b], mid, d[b]);
              #pragma unroll
              for (int b = 0; b < NB; ++b) d[b] = mma16<bf16_t>(wf[b], hi, d[b]);
              #pragma unroll
              for (int b = 0; b < NB; ++b) acc[b][t] += d[b];
            }
          };
          // one question for all tiles of the step: asked for each, its branch kept them from overlapping
          if (__builtin_expect(__any(top == __builtin_huge_valf()), 0)) multiply(DmTag<1>{}); else multiply(DmTag<0>{});
        }
      }
      if (RUNS && ((p + 1) % (DM_RUN / SPW) == 0 || p + 1 == P)) {
        #pragma unroll
        for (int b = 0; b < NB; ++b)
          #pragma unroll
          for (int t = 0; t < NT; ++t) { sum[b][t] += acc[b][t]; acc[b][t] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
      }
    }
  }

  // ---- partial sums of the math waves: part[w][b][t][lane] (16 bytes each), then the waves' shares of sum x^2
  __syncthreads();                                         // every wave has left the ring
  f32x4 *part = reinterpret_cast<f32x4 *>(dm_lds);
  float *sq = reinterpret_cast<float *>(dm_lds) + KW * NB * NT * 256;         // [KW][NT][16]
  if (wave < KW) {
    #pragma unroll
    for (int b = 0; b < NB; ++b)
      #pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f32x4 v = RUNS ? sum[b][t] : acc[b][t];
        part[((wave * NB + b) * NT + t) * 64 + lane] = (wave & 1) ? -v : v;
      }
    if (NORM) {
      #pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float v = lanes_xor32(lanes_xor16(ss[t], AddF()), AddF());
        if (g == 0) sq[(wave * NT + t) * 16 + r16] = v;
      }
    }
  }
  __syncthreads();
  // lane ln of (block, tile) holds activation row t * 16 + ln % 16 against weight rows (ln / 16) * 4 .. + 3 of the block
  auto total = [&](int b, int t, int ln) {
    f32x4 v = part[(b * NT + t) * 64 + ln];
    #pragma unroll
    for (int w = 1; w < KW; ++w) v += part[((w * NB + b) * NT + t) * 64 + ln];
    return v;
  };
  auto inv_rms = [&](int m) {
    float s = 0.f;
    #pragma unroll
    for (int w = 0; w < KW; ++w) s += sq[w * NT * 16 + m];
    return rsqrtf(s / (float)a.Kd + a.eps);
  };
  float *lg = sq + KW * NT * 16;                        // DM_LMTOPK: [NT * 16][16 * NB] logits of this workgroup

  for (int idx = tid; idx < NB * NT * 64; idx += THREADS) {
    const int ln = idx & 63, bt = idx >> 6, t = bt % NT, b = bt / NT, q = ln >> 4, m = t * 16 + (ln & 15);
    if (b0 + b > bl_last || m >= a.M) continue;
    const int blk = head * bps + b0 + b;
    if (EPI == DM_SWIGLU) {
      // lane groups 0, 1 hold the block's 8 gate rows, groups 2, 3 the same rows of W_up
      if (q >= 2) continue;
      const float rs = inv_rms(m);
      const f32x4 gt = total(b, t, ln), up = total(b, t, ln + 32);
      const int n0 = blk * 8 + q * 4;
      #pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n0 + j < a.seg_rows) a.o0[(size_t)m * a.ldo + n0 + j] = silu_f(gt[j] * rs) * (up[j] * rs);
    } else if (EPI == DM_SALQKV) {
      const int seg = blk / bps, bl = blk - seg * bps, bph = a.d_h >> 4, half = a.d_h >> 1;
      const int bb = (a.row0 + m) / a.R, jn = (a.row0 + m) % a.R;
      const bool valid = !(a.n_valid && jn >= a.n_valid[bb]);
      const int sl = a.sal_len[bb], pos = sl + jn;
      const bool bad = valid && (sl < 0 || pos + 1 > a.max_kv);
      if (bad && blk == 0 && q == 0) atomicOr(a.dev_status, 1u);
      if (!valid || bad || (seg < 2 && q >= 2)) continue;
      const float rs = inv_rms(m);
      f32x4 v = total(b, t, ln);
      bf16_t *kv = a.kv_stage + (((size_t)bb * 2 + (seg == 2 ? 1 : 0)) * a.n_heads) * (size_t)a.max_kv * a.d_h + (size_t)pos * a.d_h;
      if (seg == 2) {
        const int n = bl * 16 + q * 4;
        const float y[4] = {v[0] * rs, v[1] * rs, v[2] * rs, v[3] * rs};
        store4<bf16_t>(kv + (size_t)(n / a.d_h) * a.max_kv * a.d_h + n % a.d_h, y);
        continue;
      }
      const f32x4 v2 = total(b, t, ln + 32);
      const int hd = bl / bph, i0 = (bl % bph) * 8 + q * 4;
      float y1[4], y2[4];
      #pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float inv_freq = exp2f(-2.0f * (float)(i0 + j) / (float)a.d_h * log2f(a.theta));
        float sn, cs;
        sincosf((float)pos * inv_freq, &sn, &cs);
        const float xa = v[j] * rs, xb = v2[j] * rs;
        y1[j] = xa * cs - xb * sn;
        y2[j] = xb * cs + xa * sn;
      }
      if (seg == 0) {
        float *dst = a.o0 + (size_t)m * a.ldo + hd * a.d_h + i0;
        store4<float>(dst, y1);
        store4<float>(dst + half, y2);
      } else {
        bf16_t *dst = kv + (size_t)hd * a.max_kv * a.d_h + i0;
        store4<bf16_t>(dst, y1);
        store4<bf16_t>(dst + half, y2);
      }
    } else {
      const int seg = EPI == DM_HEADMLP ? head : (a.n_seg == 1 ? 0 : blk / bps);
      const int n0 = (blk - seg * bps) * 16 + q * 4;
      const f32x4 v = total(b, t, ln);
      if (EPI == DM_LMTOPK) {
        *reinterpret_cast<f32x4 *>(lg + m * (16 * NB) + b * 16 + q * 4) = v;
        if (a.logits) {
          #pragma unroll
          for (int j = 0; j < 4; ++j)
            if (n0 + j < a.seg_rows) a.logits[(size_t)m * a.ldo + n0 + j] = v[j];
        }
      } else if (EPI == DM_HEADMLP) {
        const float *src = ((head >= a.K / 2) ? a.x2 : a.x) + (size_t)m * a.ldx;
        #pragma unroll
        for (int j = 0; j < 4; ++j)
          if (n0 + j < a.seg_rows) {
            const float pek = a.pe ? Elem<bf16_t>::to_f32(a.pe[(size_t)head * a.ldx + n0 + j]) : 0.f;
            a.o0[((size_t)m * a.K + head) * a.ldx + n0 + j] = src[n0 + j] + silu_f(v[j]) + pek;
          }
      } else {
        if (S > 1) {                                       // partial sums, added up by k_draft_fold (seg_rows is a multiple of 4)
          if (n0 < a.seg_rows) *reinterpret_cast<f32x4 *>(a.slabs + ((size_t)blockIdx.z * a.M + m) * a.seg_rows + n0) = v;
          continue;
        }
        float *out = (seg == 0 ? a.o0 : seg == 1 ? a.o1 : a.o2) + (size_t)m * a.ldo + n0;
        const float *res = a.res ? a.res + (size_t)m * a.ldo + n0 : nullptr;
        const int last_b = last_row_of(a.last, m);
        #pragma unroll
        for (int j = 0; j < 4; ++j)
          if (n0 + j < a.seg_rows) {
            const float y = res ? v[j] + res[j] : v[j];
            out[j] = y;
            if (last_b >= 0) a.last.out[(size_t)last_b * a.ldo + n0 + j] = y;
          }
      }
    }
  }

  if (EPI == DM_LMTOPK) {
    // the k best of this workgroup's 16 * NB logits of every row (fewer in the last workgroup), as k_lmhead_topk leaves them
    __syncthreads();
    constexpr int NPT = (16 * NB + 63) / 64;
    const int n_live = min(16 * NB, a.seg_rows - b0 * 16);
    for (int m = wave; m < a.M; m += KW + DM_NL) {
      float xv[NPT];
      #pragma unroll
      for (int j = 0; j < NPT; ++j) xv[j] = lg[m * (16 * NB) + min(j * WAVE + lane, 16 * NB - 1)];
      const size_t o = ((size_t)m * gridDim.x + blockIdx.x) * a.topk;
      rank_select<NPT>(xv, b0 * 16, n_live, a.topk, a.cand_v + o, a.cand_i + o);
    }
  }
}

// out[m][n] = (res ? res[m][n] : 0) + sum_s slabs[s][m][n], s ascending; everything is requested before the first use.
template <int S>
__global__ __launch_bounds__(256) void k_draft_fold(const float *slabs, int n, const float *res, float *out, int ld, const LastRows last) {
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  const int m = i / ld, last_b = last_row_of(last, m);     // (ld is a multiple of 4)
  f32x4 v[S], r = (f32x4){0.f, 0.f, 0.f, 0.f};
  #pragma unroll
  for (int s = 0; s < S; ++s) v[s] = *reinterpret_cast<const f32x4 *>(slabs + (size_t)s * n + i);
  if (res) r = *reinterpret_cast<const f32x4 *>(res + i);
  #pragma unroll
  for (int s = 1; s < S; ++s) v[0] += v[s];
  v[0] += r;
  *reinterpret_cast<f32x4 *>(out + i) = v[0];
  if (last_b >= 0) *reinterpret_cast<f32x4 *>(last.out + (size_t)last_b * ld + (i - m * ld)) = v[0];
}

// ---- host side --------------------------------------------------------------------------------------
constexpr int DM_LDS = 160 * 1024;

template <int NB, int NT, int CB> static size_t dm_tail_bytes(bool lm) {       // LDS after the loop
  return (size_t)DmStage<NB, NT, CB>::KW * NT * (NB * 1024 + 64) + (lm ? (size_t)NT * 16 * NB * 64 : 0);
}

template <int EPI, int NB, int NT, int CB>
static hipError_t dm_launch_cb(hipStream_t st, DmArgs a, int grid_x, int grid_y, int S) {
  using C = DmStage<NB, NT, CB>;
  constexpr bool NORM = EPI == DM_SALQKV || EPI == DM_SWIGLU;
  // two workgroups share a compute unit when there are more than one per unit; otherwise one has the LDS to itself
  const size_t tail = dm_tail_bytes<NB, NT, CB>(EPI == DM_LMTOPK);
  const size_t budget = (long long)grid_x * grid_y * S > 256 ? 80 * 1024 : 160 * 1024;
  const int nx = (a.M + C::RPX - 1) / C::RPX * C::LPX;
  a.stage_bytes = C::WB + nx * 1024 + (NORM ? DM_GAIN_B : 0);
  const int loads = C::LPW + (nx + 1) / 2 + 1;             // of one loader wave and stage
  const size_t slack = (size_t)(NT * 16 - a.M) * C::XRB;  // rows past M of the last tile are read from LDS too (and dropped)
  a.ring = std::max(2, std::min((int)((budget - slack) / a.stage_bytes), std::min(DM_MAX_R, 63 / loads + 2)));
  const size_t smem = std::max((size_t)a.ring * a.stage_bytes + slack, tail);
  if (smem > (size_t)DM_LDS) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute((const void *)k_draft_mm<EPI, NB, NT, CB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_draft_mm<EPI, NB, NT, CB>), dim3(grid_x, grid_y, S), dim3(C::THREADS), smem, st, a);
  return hipGetLastError();
}

// Bytes of a row per stage: as many as still leave a ring of three stages or more.  A stage costs 0.28 us whatever it
// holds (barrier, LDS read, one chain of arithmetic) plus 0.05 us per KB (measured with 5 rows: 4096 x 11008 in stages of
// 256 / 512 bytes 43.0 / 30.6 us, 12288 x 4096 22.4 / 20.5); with two workgroups on a compute unit one's fixed part
// hides behind the other's, and the smaller stages leave the ring deep enough (22016 x 4096: 32.0 / 32.8 us).
template <int EPI, int NB, int NT>
static hipError_t dm_launch_nt(hipStream_t st, const DmArgs &a, int grid_x, int grid_y, int S) {
  const bool alone = (long long)grid_x * grid_y * S <= 256;
  if constexpr (NT == 1 && NB == 1 && EPI != DM_FC)
    if (alone) return dm_launch_cb<EPI, NB, NT, 1024>(st, a, grid_x, grid_y, S);
  if constexpr (NT == 1 && NB <= 4)
    if (NB == 1 || alone) return dm_launch_cb<EPI, NB, NT, 512>(st, a, grid_x, grid_y, S);
  return dm_launch_cb<EPI, NB, NT, 256>(st, a, grid_x, grid_y, S);
}

template <int EPI, int NB>
static hipError_t dm_launch_nb(hipStream_t st, const DmArgs &a, int grid_x, int grid_y, int S) {
  switch ((a.M + 15) / 16) {
    case 1: return dm_launch_nt<EPI, NB, 1>(st, a, grid_x, grid_y, S);
    case 2: return dm_launch_nt<EPI, NB, 2>(st, a, grid_x, grid_y, S);
    case 3: return dm_launch_nt<EPI, NB, 3>(st, a, grid_x, grid_y, S);
    default: return hipErrorInvalidValue;
  }
}

// Row blocks per workgroup and splits of the reduction axis, by a model in us (measured as above): per 256 bytes of the
// rows 0.19 per block (4 KB at a compute unit's share of the HBM rate), the activations' cutting and transfer per tile and
// row, and the stage's fixed cost where a workgroup has its compute unit to itself.  Up to two workgroups share a unit.
// (5 rows, blocks per workgroup 2 / 3 / 4 / 6: 22016 x 4096 47.1 / 32.0 / 36.7 / 38.0 us, 27648 x 5120 55.6 / 58.7 /
// 46.8 / 57.7, 35840 x 6656 91.9 / 77.9 / 88.7 / 77.5.)
// Every workgroup reads all activations of its stages, at M * 4 bytes a column against NB * 32 of weights, and a compute
// unit takes in 40 GB/s of the two together.  With many rows against few blocks that is the time; S workgroups with S
// times the blocks and 1 / S of the axis each halve or quarter it, for a fold of S slabs (4 blocks
// and 4 splits against 1 and 1, without the fold's 4.8 us: 40 rows, 4096 x 4096 34 / 16.5 us, 4096 x 11008 83 / 33, Eq. 1's
// 4096 x 8192 50 / 25; 5 rows 13.6 / 10.7, 29 / 20, 26 / 17).
struct DmPick { int nb, S; };
static DmPick dm_pick(int blocks, int groups, int M, int N, int Kd, bool lm, bool may_split) {
  static const int sizes[] = {1, 2, 3, 4, 6};
  const int nt = (M + 15) / 16;
  const double act = 0.125 * nt + 0.012 * M, chunks = Kd / 128.0;
  double best = 1e300;
  DmPick pick = {1, 1};
  for (int S = 1; S <= (may_split ? DRAFT_MM_SPLITS : 1); S *= 2) {
    if (S > 1 && Kd / S < 1024) break;
    for (int s : sizes) {
      if (lm && s != 4) continue;
      if (!lm && Kd / S > DM_LONG && s > DM_RUNS_NB) continue;
      const long wgs = (long)((blocks + s - 1) / s) * groups * S;
      const double fixed = (nt == 1 && s <= 4) ? 0.14 : 0.28;
      double cost = wgs <= 256 ? 0.19 * s + act + fixed : (double)((wgs + 511) / 512) * 2 * (0.19 * s + act);
      // two workgroups on a unit whose halves of the LDS hold only two stages each (35840 x 6656 over 24 rows: 6 blocks,
      // two stages 140 us; 3 blocks, three stages 120 us)
      if (wgs > 256 && 3 * (s * 4096 + M * 512 + 1024) > 80 * 1024) cost *= 1.35;
      cost *= chunks / S;
      if (S > 1) cost += 5.0 + 2.0e-6 * S * M * N;           // the fold's launch, the slabs' way out and back
      if (cost < best) { best = cost; pick = {s, S}; }
    }
  }
  return pick;
}

template <int EPI>
static hipError_t dm_launch(hipStream_t st, DmArgs a, int blocks, int groups) {
  if (a.M < 1 || a.M > DRAFT_MM_ROWS || a.Kd < 8 || a.Kd % 8) return hipErrorInvalidValue;
  a.blocks = blocks;
  const bool may_split = (EPI == DM_LINEAR || EPI == DM_FC) && a.slabs && a.n_seg == 1 && a.seg_rows % 4 == 0 && a.ldo == a.seg_rows;
  const DmPick p = dm_pick(blocks, groups, a.M, a.seg_rows, a.Kd, EPI == DM_LMTOPK, may_split);
  const int gx = (blocks + p.nb - 1) / p.nb;
  hipError_t e;
  if constexpr (EPI == DM_LMTOPK) e = dm_launch_nb<EPI, 4>(st, a, gx, groups, 1);
  else switch (p.nb) {
    case 1: e = dm_launch_nb<EPI, 1>(st, a, gx, groups, p.S); break;
    case 2: e = dm_launch_nb<EPI, 2>(st, a, gx, groups, p.S); break;
    case 3: e = dm_launch_nb<EPI, 3>(st, a, gx, groups, p.S); break;
    case 4: e = dm_launch_nb<EPI, 4>(st, a, gx, groups, p.S); break;
    default: e = dm_launch_nb<EPI, 6>(st, a, gx, groups, p.S); break;
  }
  if (e != hipSuccess || p.S == 1) return e;
  const int n = a.M * a.seg_rows;
  const dim3 grid((n / 4 + 255) / 256), block(256);
  static_assert(DRAFT_MM_SPLITS == 4, "the folds below");
  if (p.S == 2) hipLaunchKernelGGL((k_draft_fold<2>), grid, block, 0, st, a.slabs, n, a.res, a.o0, a.ldo, a.last);
  else hipLaunchKernelGGL((k_draft_fold<4>), grid, block, 0, st, a.slabs, n, a.res, a.o0, a.ldo, a.last);
  return hipGetLastError();
}

hipError_t draft_mm_fc(hipStream_t st, const void *W, const float *u, const void *embed, const int32_t *tok, int vocab, int d, int M,
                       float *out, uint32_t *dev_status, float *slabs, const LastRows &last) {
  if (d % 256) return hipErrorInvalidValue;               // a stage holds columns of one half of the concatenated row only
  DmArgs a{};
  a.w0 = (const bf16_t *)W; a.n_seg = 1; a.seg_rows = d; a.Kd = 2 * d; a.M = M; a.x = u; a.ldx = d; a.o0 = out; a.ldo = d;
  a.embed = (const bf16_t *)embed; a.tok = tok; a.vocab = vocab; a.dev_status = dev_status; a.slabs = slabs;
  a.last = last;
  return dm_launch<DM_FC>(st, a, (d + 15) / 16, 1);
}

hipError_t draft_mm_sal_qkv(hipStream_t st, const amph_layer_w &lw, const float *x, int d, int n_heads, int d_h, int M, float eps,
                            float theta, const int32_t *sal_len, int max_kv, void *kv_stage, float *qbuf, uint32_t *dev_status,
                            int row0, int R, const int32_t *n_valid) {
  if (d % 16 || d_h % 16) return hipErrorInvalidValue;
  DmArgs a{};
  a.w0 = (const bf16_t *)lw.wq; a.w1 = (const bf16_t *)lw.wk; a.w2 = (const bf16_t *)lw.wv;
  a.n_seg = 3; a.seg_rows = d; a.Kd = d; a.M = M; a.x = x; a.ldx = d; a.gain = (const bf16_t *)lw.rms1; a.eps = eps;
  a.o0 = qbuf; a.ldo = d; a.n_heads = n_heads; a.d_h = d_h; a.max_kv = max_kv; a.row0 = row0; a.R = R; a.theta = theta;
  a.sal_len = sal_len; a.n_valid = n_valid; a.kv_stage = (bf16_t *)kv_stage; a.dev_status = dev_status;
  return dm_launch<DM_SALQKV>(st, a, 3 * (d / 16), 1);
}

hipError_t draft_mm_linear(hipStream_t st, const void *w0, const void *w1, const void *w2, int n_seg, int seg_rows, int Kd,
                           const float *x, int ldx, int M, const float *res, float *o0, float *o1, float *o2, int ldo, float *slabs,
                           const LastRows &last) {
  DmArgs a{};
  a.w0 = (const bf16_t *)w0; a.w1 = (const bf16_t *)w1; a.w2 = (const bf16_t *)w2; a.n_seg = n_seg; a.seg_rows = seg_rows; a.Kd = Kd;
  a.M = M; a.x = x; a.ldx = ldx; a.res = res; a.o0 = o0; a.o1 = o1; a.o2 = o2; a.ldo = ldo; a.slabs = slabs; a.last = last;
  return dm_launch<DM_LINEAR>(st, a, n_seg * ((seg_rows + 15) / 16), 1);
}

hipError_t draft_mm_gate_up(hipStream_t st, const amph_layer_w &lw, const float *x, int d, int f, int M, float eps, float *act) {
  DmArgs a{};
  a.w0 = (const bf16_t *)lw.w_gate; a.w1 = (const bf16_t *)lw.w_up; a.n_seg = 2; a.seg_rows = f; a.Kd = d; a.M = M; a.x = x; a.ldx = d;
  a.gain = (const bf16_t *)lw.rms2; a.eps = eps; a.o0 = act; a.ldo = f;
  return dm_launch<DM_SWIGLU>(st, a, (f + 7) / 8, 1);
}

hipError_t draft_mm_head_mlp(hipStream_t st, const void *w_mlp, const void *pe, const float *h1, const float *h2, int d, int K, int M,
                             float *Hp) {
  DmArgs a{};
  a.w0 = (const bf16_t *)w_mlp; a.n_seg = K; a.seg_rows = d; a.Kd = d; a.M = M; a.x = h1; a.x2 = h2; a.ldx = d; a.pe = (const bf16_t *)pe;
  a.K = K; a.o0 = Hp;
  return dm_launch<DM_HEADMLP>(st, a, (d + 15) / 16, K);
}

int draft_mm_lmhead_wgs(int V) { return ((V + 15) / 16 + 3) / 4; }

hipError_t draft_mm_lmhead(hipStream_t st, const void *W, int V, int Kd, const float *x, int M, int k, float *logits, float *cand_v,
                           int *cand_i) {
  DmArgs a{};
  a.w0 = (const bf16_t *)W; a.n_seg = 1; a.seg_rows = V; a.Kd = Kd; a.M = M; a.x = x; a.ldx = Kd; a.ldo = V;
  a.logits = logits; a.cand_v = cand_v; a.cand_i = cand_i; a.topk = k;
  return dm_launch<DM_LMTOPK>(st, a, (V + 15) / 16, 1);
}

}  // namespace amph

// GEMMs of the target's forward pass over the tree tokens (Sec. 2 "Tree Attention"): M = B*T activation rows
// against [N, Kd] weights that stream from HBM once, on the matrix cores.  Two kernels: the skinny one
// (described first; up to 64 rows, or row-major weights) and the wide one (further down; more than 128 rows, and most
// matrices from 65 on).
//
// The unit of work is a ROW BLOCK: 16 weight rows that one wave keeps as matrix-core A fragments and
// whose outputs need nothing from any other block:
//   * plain / LM head: rows 16b .. 16b+15;
//   * q and k: 8 rows of a head and their 8 RoPE partners (i, i + d_h/2); v: 16 consecutive rows
//     (blocks numbered q, then k, then v);
//   * gate/up: rows 8b .. 8b+7 of W_gate and the same rows of W_up.
// A workgroup owns nb consecutive blocks (a 64 x 16*nb output tile) and a slice of the reduction axis,
// and its waves have two roles:
//   * nb math waves, one block each.  Their A fragments are 16-byte loads straight from global memory,
//     requested one 512-byte chunk (8 fragments) ahead; B fragments come from LDS.  They issue nothing
//     else, so waiting for a chunk of weights never waits for anything younger.
//   * 4 loader waves, which bring the activations of each chunk (64 rows x 512 bytes, L2 hits) into a
//     padded, double-buffered LDS tile one chunk ahead.
// One barrier per chunk joins the two.  nb (2..12) and the split of the reduction axis are chosen per
// shape by gemm_plan: every workgroup reads the whole activation slice from L2, so that traffic is
// (64 / tile height) times the weight bytes and measurably slows the weight stream; taller tiles cut
// it as far as filling the 256 CUs in whole rounds allows.
//
// Weight layouts.  Row-major [N, Kd] works, but a matrix-core A fragment is 16 rows x 64 bytes, so
// every wave load touches 16 half cache lines; the vector L1 handles such loads at about a quarter of
// the rate of a contiguous 1 KB load and the weight stream then stalls on the CU side, not on HBM
// (measured: 41 us against 33 us for the gate/up shape).  The tiled layout (k_pack_weights, run once
// per matrix) stores every fragment as one contiguous 1 KB piece, block-major:
//   tiled[(block * (Kd * sizeof(T) / 64) + step) * 1024 + r * 64 + byte]  =  W[row(block, r)][step * 64 + byte]
// with rows past N stored as zeros.
//
// No workgroup ever communicates with another inside the kernel (a device-scope fence per workgroup
// costs far more than the kernel on this chip): a split reduction axis writes one partial slab per
// split, which the consumer (the RMSNorm kernel of the next sub-layer, or k_sum_slabs) adds up in a
// fixed order; per-tile argmax candidates are folded by k_argmax_fold.  Fused epilogues: RoPE from a
// precomputed table + KV-cache write, SwiGLU, per-tile row argmax.
#include "kernels.h"
#include <hip/hip_ext.h>
#include <algorithm>

namespace amph {

constexpr int GM_BM = 64;
constexpr int GM_CHUNK_B = 512;                 // bytes of one activation row per chunk
constexpr int GM_PITCH = GM_CHUNK_B + 16;       // LDS row pitch (bytes): rows shift by 4 banks
constexpr int GM_STEPS = GM_CHUNK_B / 64;       // matrix-core steps per chunk (64 bytes of k each)
constexpr int GM_STAGE = GM_BM * GM_PITCH;      // one activation stage
constexpr int GM_LDS_BYTES = 2 * GM_STAGE;
constexpr int GM_NLW = 4;                       // loader waves
constexpr int GM_XROWS = GM_BM / GM_NLW, GM_XL = GM_XROWS / 2;   // activation rows / 16-byte loads per loader lane per chunk
constexpr int GM_MIN_NB = 2, GM_MAX_NB = 12;    // math waves (= row blocks) per workgroup
static_assert(GM_LDS_BYTES >= GM_BM * (16 * GM_MAX_NB + 4) * 4, "output tile must fit in the staging buffers");
static_assert(64 * (GM_MAX_NB + GM_NLW) <= 1024, "workgroup size");

// number of row blocks of a GEMM
__host__ __device__ inline int gemm_blocks(int epi, int seg_rows) {
  if (epi == EPI_QKV_ROPE) return 3 * (seg_rows / 16);
  if (epi == EPI_SWIGLU) return (seg_rows + 7) / 8;
  return (seg_rows + 15) / 16;
}

// weight row (within its matrix) and matrix index of row r16 of block b
struct RowMap { int seg; int n; bool valid; };

template <int EPI>
__device__ __forceinline__ RowMap map_block(const GemmArgs &a, int b, int r16) {
  RowMap o;
  if (EPI == EPI_QKV_ROPE) {
    const int d = a.n_heads * a.d_h, bps = d / 16, bph = a.d_h / 16;
    o.valid = true;
    o.seg = b / bps;
    const int bl = b % bps;
    if (o.seg < 2) o.n = (bl / bph) * a.d_h + (bl % bph) * 8 + (r16 & 7) + ((r16 >= 8) ? a.d_h / 2 : 0);
    else o.n = bl * 16 + r16;
  } else if (EPI == EPI_SWIGLU) {
    o.seg = (r16 >= 8) ? 1 : 0;
    o.n = b * 8 + (r16 & 7);
    o.valid = o.n < a.seg_rows;
  } else {
    o.seg = 0;
    o.n = b * 16 + r16;
    o.valid = o.n < a.seg_rows;
  }
  return o;
}

// A dimension and its RoPE partner, rotated.  The two products that are rounded on their own are named, and hidden from the compiler,
// which otherwise contracts now one and now the other product of a sum: a row's bits must not depend on where it is computed.
__device__ __forceinline__ void rope_pair(float x1, float x2, float cs, float sn, float &y1, float &y2) {
  float p1 = x2 * sn, p2 = x1 * sn;
  asm("" : "+v"(p1));
  asm("" : "+v"(p2));
  y1 = fmaf(x1, cs, -p1);
  y2 = fmaf(x2, cs, p2);
}

// Epilogue of one 64-row block of a workgroup's output tile: Ct[m][r] (float32, pitch CT_PITCH) holds rows
// m_base .. m_base + 63 of the activations against the tile's nb row blocks (BN = 16 * nb columns).  Every thread
// of the workgroup (NT of them) takes part.
template <typename T, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &a, const float *Ct, int CT_PITCH, int tile, int nb, int m_base,
                                              int split, int nblk, int tid, int NT) {
  constexpr int rows = GM_BM;
  const int BN = 16 * nb;
  if (EPI == EPI_STORE) {
    // out is [split_k][M][N]: slab `split` receives this workgroup's partial sums
    const int N = a.seg_rows;
    float *slab = a.out + (size_t)split * a.M * N;
    const int Q = BN / 4;                                   // 4 adjacent columns per thread (N is no multiple of 4: one by one)
    for (int idx = tid; idx < rows * Q; idx += NT) {
      const int m = idx / Q, r = (idx % Q) * 4, mg = m_base + m, n = tile * BN + r;
      if (mg >= a.M || n >= N) continue;
      for (int c = 0; c < 4 && n + c < N; ++c) slab[(size_t)mg * N + n + c] = Ct[m * CT_PITCH + r + c];
    }
  } else if (EPI == EPI_SWIGLU) {
    // block w of the tile: columns 0..7 = gate rows, 8..15 = the same rows of up
    const int f = a.seg_rows, H = 8 * nb;
    T *act = (T *)a.act;
    // one (token, block) per thread: 8 adjacent outputs
    for (int idx = tid; idx < rows * nb; idx += NT) {
      const int m = idx / nb, w = idx % nb, mg = m_base + m, j0 = tile * H + w * 8;
      if (mg >= a.M || j0 >= f) continue;
      const float *crow = Ct + m * CT_PITCH + w * 16;
      float y[8];
      #pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = silu_f(crow[j]) * crow[8 + j];
      T *dst = act + (size_t)mg * f + j0;
      for (int j = 0; j < 8 && j0 + j < f; ++j) dst[j] = Elem<T>::from_f32(y[j]);      // (f is no multiple of 4)
    }
  } else if (EPI == EPI_QKV_ROPE) {
    // d_h is a power of two (checked at launch): heads and dims come from shifts; the segment of a block (q, k or v:
    // bps blocks each) from two comparisons instead of a division by a run-time value
    const int d_h = a.d_h, d = a.n_heads * d_h, bps = d >> 4, bph = d_h >> 4, bsh = __ffs(bph) - 1, half = d_h >> 1;
    auto seg_of = [&](int b) { return (b >= 2 * bps) ? 2 : (b >= bps) ? 1 : 0; };
    // q and k blocks: one (block, token) per thread = 8 rotation pairs.  Everything the item needs from global
    // memory (64 bytes of the cos/sin table, the committed length) is requested first, for up to QK_U items of the
    // thread at once: stores in between would keep the next item's loads from starting early.  The 8 + 8 results leave as 16-byte pieces: dims e0 .. e0+7 (and their partners at
    // + d_h/2) are adjacent in q and inside a fragment of the tiled K cache.
    constexpr int QK_U = 3;
    for (int base = tid; base < nb * rows; base += QK_U * NT) {
      float4 tab[QK_U][4];
      int Lb[QK_U];
      #pragma unroll
      for (int u = 0; u < QK_U; ++u) {
        const int idx = base + u * NT, w = idx / rows, m = idx % rows, b = tile * nb + w, mg = m_base + m;
        const bool live = idx < nb * rows && b < nblk && mg < a.M && seg_of(b) < 2;
        const int e0 = ((b - seg_of(b) * bps) & (bph - 1)) * 8;
        // (unconditional loads from clamped addresses: dead items read the table's first entry and element 0's length)
        const float4 *csp = reinterpret_cast<const float4 *>(a.rope_cs + (live ? (size_t)mg * half + e0 : (size_t)0));
        #pragma unroll
        for (int k = 0; k < 4; ++k) tab[u][k] = csp[k];
        Lb[u] = a.kv_len[live ? mg / a.T_nodes : 0];
      }
      #pragma unroll
      for (int u = 0; u < QK_U; ++u) {
        const int idx = base + u * NT, w = idx / rows, m = idx % rows, b = tile * nb + w, mg = m_base + m;
        if (idx >= nb * rows || b >= nblk || mg >= a.M) continue;
        const int seg = seg_of(b), bl = b - seg * bps;
        if (seg >= 2) continue;
        const int head = bl >> bsh, e0 = (bl & (bph - 1)) * 8;
        const float4 c01 = tab[u][0], c23 = tab[u][1], c45 = tab[u][2], c67 = tab[u][3];
        const float cs[8] = {c01.x, c01.z, c23.x, c23.z, c45.x, c45.z, c67.x, c67.z};
        const float sn[8] = {c01.y, c01.w, c23.y, c23.w, c45.y, c45.w, c67.y, c67.w};
        const float *crow = Ct + m * CT_PITCH + w * 16;
        float y1[8], y2[8];
        #pragma unroll
        for (int j = 0; j < 8; ++j) {
          rope_pair(crow[j], crow[8 + j], cs[j], sn[j], y1[j], y2[j]);
        }
        T *dst1, *dst2;
        if (seg == 0) {
          dst1 = (T *)a.q_out + (size_t)mg * d + head * d_h + e0;
          dst2 = dst1 + half;
        } else {
          const int bb = mg / a.T_nodes, node = mg % a.T_nodes, L = Lb[u];
          if (L < 0 || L + a.T_nodes > a.max_kv) {
            if (node == 0 && e0 == 0) atomicOr(a.dev_status, 2u);
            continue;
          }
          T *kc = (T *)a.k_cache + ((size_t)bb * a.n_heads + head) * (size_t)a.max_kv * d_h;
          dst1 = kc + k_tiled_index<T>(L + node, e0, d_h);
          dst2 = kc + k_tiled_index<T>(L + node, e0 + half, d_h);
        }
        store4<T>(dst1, y1); store4<T>(dst1 + 4, y1 + 4);
        store4<T>(dst2, y2); store4<T>(dst2 + 4, y2 + 4);
      }
    }
    // v blocks: a thread takes 8 of a block's 16 dims for one token.  rows divides the number of threads, so a thread keeps
    // its token through the loop: its committed length is read once, ahead of the stores, and consecutive threads write
    // consecutive tree rows, which are adjacent inside a step-tiled piece.  A block's dims are adjacent pieces, so its
    // addresses are one base and constants (computed for each element they took longer than the stores).
    {
      constexpr int PIECE = 64 / (int)sizeof(T);
      const int m = tid % rows, mg = m_base + m;
      const bool row_ok = mg < a.M;
      const int bb = row_ok ? mg / a.T_nodes : 0, node = row_ok ? mg % a.T_nodes : 0;
      const int L = a.kv_len[bb];
      if (row_ok && L >= 0 && L + a.T_nodes <= a.max_kv) {
        T *vb = (T *)a.v_cache + (size_t)bb * a.n_heads * (size_t)a.max_kv * d_h;
        const size_t at = v_tiled_index<T>(L + node, 0, d_h);
        for (int q = tid / rows; q < nb * 2; q += NT / rows) {
          const int w = q >> 1, hh = q & 1, b = tile * nb + w, bl = b - 2 * bps;
          if (b >= nblk || bl < 0) continue;
          T *dst = vb + (size_t)(bl >> bsh) * (size_t)a.max_kv * d_h + at + ((bl & (bph - 1)) * 16 + hh * 8) * PIECE;
          const float *c = Ct + m * CT_PITCH + w * 16 + hh * 8;
          #pragma unroll
          for (int j = 0; j < 8; ++j) dst[j * PIECE] = Elem<T>::from_f32(c[j]);
        }
      }
    }
  }
}

// the best (value, column) of the four lane groups of 16, in every lane
__device__ __forceinline__ void best_of_groups(float &bv, int &bi) {
  const auto ov = __builtin_amdgcn_permlane16_swap(lane_bits(bv), lane_bits(bv), false, false);
  const auto oi = __builtin_amdgcn_permlane16_swap((unsigned)bi, (unsigned)bi, false, false);
  bv = lane_value<float>(ov[0]); bi = (int)oi[0];
  take_better(bv, bi, lane_value<float>(ov[1]), (int)oi[1]);
  const auto pv = __builtin_amdgcn_permlane32_swap(lane_bits(bv), lane_bits(bv), false, false);
  const auto pi = __builtin_amdgcn_permlane32_swap((unsigned)bi, (unsigned)bi, false, false);
  bv = lane_value<float>(pv[0]); bi = (int)pi[0];
  take_better(bv, bi, lane_value<float>(pv[1]), (int)pi[1]);
}

template <int N> struct GemmTag { static constexpr int value = N; };

template <typename T, int EPI, bool TILED>
__global__ __launch_bounds__(64 * (GM_MAX_NB + GM_NLW)) void k_gemm_skinny(const GemmArgs a, int tiles) {
  __shared__ __align__(16) unsigned char lds[GM_LDS_BYTES];
  const int nb = a.nb, BN = 16 * nb, NT = 64 * (nb + GM_NLW), CT_PITCH = BN + 4;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  const int S = a.split_k;
  // Workgroup index -> (unit = tile and split, block of 64 activation rows).  With more than one row block
  // the workgroups that stream the SAME weights get indices 8 apart: they are dispatched together and
  // land on the same XCD, so the weights come from HBM once and from that XCD's L2 for the others.
  const int mblocks = (a.M + GM_BM - 1) / GM_BM;
  const int id = blockIdx.x, unit = (id / 8 / mblocks) * 8 + (id & 7), mblock = (id / 8) % mblocks;
  if (unit >= tiles * S) return;                          // padding of the last group of 8 units (whole workgroup)
  const int tile = unit / S, split = unit % S;
  const int m_base = mblock * GM_BM;
  const int row_bytes = a.Kd * (int)sizeof(T);
  const int total_steps = row_bytes / 64;
  const int ssh = __ffs(S) - 1;                           // S is 1, 2, 4 or 8
  const int s0 = (total_steps * split) >> ssh, s1 = (total_steps * (split + 1)) >> ssh;
  const int nch = (s1 - s0 + GM_STEPS - 1) / GM_STEPS;
  const int nblk = gemm_blocks(EPI, a.seg_rows);
  // Both roles run the same number of iterations (a multiple of two, the depth of every ring) with
  // no conditional inside: chunks past the slice load clamped addresses and stage zeros, so the
  // compiler can count outstanding loads exactly instead of draining them at every join.
  const int nch2 = (nch + 1) & ~1;

  f32x4 acc[4];
  #pragma unroll
  for (int mb = 0; mb < 4; ++mb) acc[mb] = (f32x4){0.f, 0.f, 0.f, 0.f};

  if (wave < nb) {
    // ------------------------------------------------------------------------------- math wave
    // A block past the end (last tile only) re-reads the last block; its results are never stored.
    const int blk = min(tile * nb + wave, nblk - 1);
    const unsigned char *wrow;
    if (TILED) {
      // the block's fragments lie one after another: step st is the 1 KB at st * 1024, this lane's 16 bytes at
      // (r16 * 64 + g * 16) inside it
      wrow = (const unsigned char *)a.wt + (size_t)blk * total_steps * 1024 + r16 * 64 + g * 16;
    } else {
      const RowMap rm = map_block<EPI>(a, blk, r16);
      const void *wm = (rm.seg == 0) ? a.w0 : (rm.seg == 1) ? a.w1 : a.w2;
      wrow = (const unsigned char *)wm + (size_t)(rm.valid ? rm.n : 0) * row_bytes + g * 16;
    }
    uint4 aw[2][GM_STEPS];
    auto load_w = [&](int c, uint4 (&af)[GM_STEPS]) {
      #pragma unroll
      for (int s = 0; s < GM_STEPS; ++s) {
        // Unconditional load (a predicated load with a zero alternative makes the compiler wait for every
        // load at the merge).  Steps past the slice re-read its last step: harmless, because the activation
        // tile is zero there and weights are finite; rows past N re-read row 0 and are never stored.
        const int st = min(s0 + c * GM_STEPS + s, s1 - 1);
        af[s] = ldg16_stream(wrow + (size_t)st * (TILED ? 1024 : 64));
      }
    };
    load_w(0, aw[0]);
    __syncthreads();
    // Only the 16-row tiles that hold rows of the call are multiplied: in float32 a tile is 128 clocks of matrix core per
    // step, which is what a small tree's launch lasts (16 rows, us: QKV 768 x 256 9.6 -> 6.9, 256 x 688 12.9 -> 7.3).
    auto run = [&](auto tag) {
      constexpr int MB = decltype(tag)::value;
      for (int c = 0; c < nch2; c += 2) {
        #pragma unroll
        for (int u = 0; u < 2; ++u) {
          load_w(c + u + 1, aw[u ^ 1]);
          const unsigned char *buf = lds + u * GM_STAGE;
          #pragma unroll
          for (int s = 0; s < GM_STEPS; ++s) {
            #pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
              const uint4 bfrag = *reinterpret_cast<const uint4 *>(buf + (mb * 16 + r16) * GM_PITCH + s * 64 + g * 16);
              acc[mb] = mma16<T>(aw[u][s], bfrag, acc[mb]);
            }
          }
          __syncthreads();
        }
      }
    };
    // In bf16 a tile is 16 clocks a step and the weights set the pace.
    if (sizeof(T) == 2) run(GemmTag<4>{});
    else switch ((min(a.M - m_base, GM_BM) + 15) / 16) {    // (uniform)
      case 1: run(GemmTag<1>{}); break;
      case 2: run(GemmTag<2>{}); break;
      case 3: run(GemmTag<3>{}); break;
      default: run(GemmTag<4>{}); break;
    }
  } else {
    // ----------------------------------------------------------------------------- loader wave
    // 32 lanes cover one 512-byte row piece, a wave instruction two rows; chunk c+1 is written to its
    // stage while the math waves work on chunk c, and chunk c+2 is already on its way from L2.
    const unsigned char *xg = (const unsigned char *)a.x;
    const int x_row0 = (wave - nb) * GM_XROWS + (lane >> 5), x_col = (lane & 31) * 16;
    uint4 xr[2][GM_XL];
    auto load_x = [&](int c, uint4 (&xf)[GM_XL]) {
      const int byte = (s0 + c * GM_STEPS) * 64 + x_col;
      const bool in_k = byte < s1 * 64;
      #pragma unroll
      for (int j = 0; j < GM_XL; ++j) {
        const int mg = m_base + x_row0 + 2 * j;
        const bool ok = in_k && mg < a.M;                 // out-of-range pieces read the tensor's first bytes ...
        xf[j] = ldg16(xg + (ok ? (size_t)mg * row_bytes + byte : (size_t)0));
      }
    };
    auto store_x = [&](int stage, int c, const uint4 (&xf)[GM_XL]) {
      unsigned char *buf = lds + stage * GM_STAGE;
      const bool in_k = (s0 + c * GM_STEPS) * 64 + x_col < s1 * 64;
      #pragma unroll
      for (int j = 0; j < GM_XL; ++j) {
        const bool ok = in_k && (m_base + x_row0 + 2 * j) < a.M;   // ... and are replaced by zeros here
        *reinterpret_cast<uint4 *>(buf + (x_row0 + 2 * j) * GM_PITCH + x_col) = ok ? xf[j] : make_uint4(0u, 0u, 0u, 0u);
      }
    };
    load_x(0, xr[0]);
    load_x(1, xr[1]);
    store_x(0, 0, xr[0]);
    __syncthreads();
    for (int c = 0; c < nch2; c += 2) {
      #pragma unroll
      for (int u = 0; u < 2; ++u) {
        load_x(c + u + 2, xr[u]);                         // slot of chunk c+u: already in LDS
        store_x(u ^ 1, c + u + 1, xr[u ^ 1]);
        __syncthreads();
      }
    }
  }

  // Partial slabs need no regrouping: a math lane holds 4 adjacent outputs (weight rows wave*16 + g*4 .. +3) of
  // activation row mb*16 + r16, which are 16 adjacent bytes of out[split][m][n].
  if (EPI == EPI_STORE && (a.seg_rows & 3) == 0) {
    if (wave < nb) {
      const int N = a.seg_rows, n0 = tile * BN + wave * 16 + g * 4;
      float *slab = a.out + (size_t)split * a.M * N + n0;
      #pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const int mg = m_base + mb * 16 + r16;
        if (mg < a.M && n0 < N) *reinterpret_cast<f32x4 *>(slab + (size_t)mg * N) = acc[mb];
      }
    }
    return;
  }
  // SwiGLU needs no regrouping either: lane groups 0, 1 hold the block's 8 gate rows, groups 2, 3 the same rows of
  // W_up, 32 lanes further on; after one exchange a lane of group 0 or 1 owns 4 adjacent outputs of its token.
  if (EPI == EPI_SWIGLU && (a.seg_rows & 3) == 0) {
    if (wave < nb) {
      const int f = a.seg_rows, j0 = tile * 8 * nb + wave * 8 + g * 4;
      T *act = (T *)a.act;
      #pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        float y[4];
        #pragma unroll
        for (int c = 0; c < 4; ++c) {
          const auto halves = __builtin_amdgcn_permlane32_swap(lane_bits(acc[mb][c]), lane_bits(acc[mb][c]), false, false);
          const float up = lane_value<float>(halves[1]);   // the upper half's value
          y[c] = silu_f(acc[mb][c]) * up;
        }
        const int mg = m_base + mb * 16 + r16;
        if (g < 2 && mg < a.M && j0 < f) store4<T>(act + (size_t)mg * f + j0, y);
      }
    }
    return;
  }
  // Neither does the row argmax, nor its logits: each math wave leaves the best of its 16 columns for every row, and the waves'
  // winners are compared.  (Through a tile in LDS, a float at a time: the LM head 32000 x 4096 with logits 57 us.)
  if (EPI == EPI_ARGMAX) {
    const int N = a.seg_rows, n0 = tile * BN + wave * 16 + g * 4;
    float *best_v = reinterpret_cast<float *>(lds);        // [wave][64 rows]
    int *best_i = reinterpret_cast<int *>(lds) + GM_MAX_NB * GM_BM;
    if (wave < nb) {
      const bool pieces = (N & 3) == 0 && ((uintptr_t)a.logits & 15) == 0;
      #pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const int mg = m_base + mb * 16 + r16;
        if (a.logits && mg < a.M) {                        // (a caller's logits may begin anywhere)
          float *dst = a.logits + (size_t)mg * N + n0;
          if (pieces && n0 < N) {
            *reinterpret_cast<f32x4 *>(dst) = acc[mb];
          } else {
            #pragma unroll
            for (int i = 0; i < 4; ++i) if (n0 + i < N) dst[i] = acc[mb][i];
          }
        }
        float bv = -__builtin_huge_valf(); int bi = 0x7fffffff;
        #pragma unroll
        for (int i = 3; i >= 0; --i)                       // descending: at equal values the lower column comes later
          if (n0 + i < N && acc[mb][i] >= bv) { bv = acc[mb][i]; bi = n0 + i; }
        best_of_groups(bv, bi);
        if (g == 0) { best_v[wave * GM_BM + mb * 16 + r16] = bv; best_i[wave * GM_BM + mb * 16 + r16] = bi; }
      }
    }
    __syncthreads();
    if (tid < GM_BM && m_base + tid < a.M) {
      float bv = best_v[tid]; int bi = best_i[tid];
      for (int w = 1; w < nb; ++w) take_better(bv, bi, best_v[w * GM_BM + tid], best_i[w * GM_BM + tid]);
      a.amax_val[(size_t)tile * a.M + m_base + tid] = bv;
      a.amax_idx[(size_t)tile * a.M + m_base + tid] = bi;
    }
    return;
  }
  // accumulators -> Ct[m][r] (float32): a math lane holds rows r = wave*16 + g*4 .. +4 of column m.
  // The last barrier of the loop has passed, so nobody reads the stages any more; the one write still
  // outstanding (the loaders' zero chunk nch2) went to stage nch2 % 2 before that barrier.
  float *Ct = reinterpret_cast<float *>(lds);
  if (wave < nb) {
    #pragma unroll
    for (int mb = 0; mb < 4; ++mb)
      *reinterpret_cast<f32x4 *>(Ct + (mb * 16 + r16) * CT_PITCH + wave * 16 + g * 4) = acc[mb];
  }
  __syncthreads();

  gemm_epilogue<T, EPI>(a, Ct, CT_PITCH, tile, nb, m_base, split, nblk, tid, NT);
}

// =====================================================================================================
// Wide GEMM: more than 64 activation rows (batches of trees, wide trees; gemm_is_wide).  The skinny kernel above re-reads the
// weights from L2 once per block of 64 rows, and every math wave re-reads the whole activation chunk from LDS: with several
// blocks of rows L2 and LDS, not HBM, set the pace.  Here a workgroup of four waves, one for each SIMD, owns a group of gt <= 12 tiles
// of 32 activation rows against NB = 2 NP weight row blocks; a wave owns up to six sixteens of the rows, dealt one by one, against all
// blocks (dealt as tiles of 32, two of four waves had half the work where a group has five, six, nine or ten: the target pass over
// 384 rows at 33B widths, QKV, W_o and W_down in groups of six, 678 -> 660 us).
//   * The weights are the shared operand: of every block of a stage (4 steps of 64 bytes of k) a wave brings in one step, through
//     registers (requested a stage ahead) into one of two LDS slots.
//   * The activations go from global memory (L2 hits) straight into the registers of the one wave that needs them, 3 steps ahead.
//   * A half-step is one step against half of the blocks: a weight fragment is read from LDS for the 16 x 16 matrix instructions of
//     all the wave's rows.  The fragments of the next half-step are read, the activations requested and the next stage written
//     between these instructions, in an order laid down by hand; the barrier lies ahead of a stage's last half-step, whose operands
//     are in registers by then, and the next stage's first fragments are read behind it, so that it costs nothing either.
// Why four waves: with one wave a SIMD its 512 registers hold up to 64 accumulators of 16 x 16, so an LDS fragment is used for four
// or six of them and the rows of a group are read again once for up to 16 blocks.
// Why 16 x 16 x 32 and not 32 x 32 x 16: both run at the same rate (16.7 and 16.2 clocks a 16 x 16 x 32 of work), but over the whole
// chip and on normally distributed values the clock is what the power allows, and that is more for the smaller one: 1.97 PFLOP/s
// (2.14 GHz) against 1.79 (1.86 GHz) for endless instructions on registers.  (An earlier measurement had the smaller one at half the
// rate: the compiler had put copies of accumulators between them, see gw_mma.)
// What bounds it: matrix instructions are in flight for 64 to 71 % of a large shape's clocks (46 to 55 % of QKV's and W_o's), at a clock of
// 1.8 to 2.0 GHz that the power sets; the rest is waiting for LDS reads and loads.  Small shapes wait for the weight stream.
// Measured alone, sustained (us, 32 x 32 instructions with an epilogue through LDS / now; gate/up, W_down, W_o, LM head): 7B over 256 rows
// 56 / 52, 39 / 39, 17 / 17, 69 / 65; over 512 rows 88 / 81 (1.14 PFLOP/s), 56 / 52, 28 / 28, 116 / 106 (1.27); 33B over 384 rows 166 / 152
// (1.21), 108 / 102, 45 / 43, 145 / 132; 13B over 128 rows 61 / 59, 34 / 34, 20 / 20, 61 / 61.  QKV as the plain product of its shape: 37 / 36 (7B,
// 256), 54 / 51 (512), 111 / 101 (33B), 40 / 40 (13B).
// Tried: weights two stages ahead, activations 7.5 steps ahead (more registers, no gain); five pairs and more with a tile a
// wave (LDS-bound).
// The activations must be tiled to match (a fragment gathered from row-major rows is the slow many-half-lines load): k_tile_rows
// rewrites [M, Kd] in the order of xt_index, rows past M as zeros (a few microseconds).
// =====================================================================================================
constexpr int GW_W = 4;            // waves, one per SIMD
constexpr int GW_ST = 4;           // steps (64 bytes of k) per weight stage
constexpr int GW_MAX_TW = 3;       // tiles of 32 activation rows per wave

// pairs of weight row blocks that are built for tw tiles a wave (float32, bound by its matrix cores at any tile: two sizes, two tiles at most)
constexpr bool gw_built(int elem_bytes, int np, int tw) {
  if (elem_bytes == 4) return tw <= 2 && (np == 2 || np == 4);
  return np >= 2 && (np <= 5 || (tw == 2 && (np == 6 || np == 8)));
}
constexpr int GW_MAX_NP = 8;

template <typename T>
__global__ __launch_bounds__(256) void k_tile_rows(const unsigned char *x, int M, int row_bytes, int m32_tiles, unsigned char *xt) {
  const int m16_tiles = 2 * m32_tiles;
  const size_t pieces = (size_t)(row_bytes / 64) * m16_tiles * 64;
  for (size_t p = (size_t)blockIdx.x * 256 + threadIdx.x; p < pieces; p += (size_t)gridDim.x * 256) {
    const int lane = (int)(p & 63);
    const size_t frag = p >> 6;
    const int m = (int)(frag % m16_tiles) * 16 + (lane & 15), st = (int)(frag / m16_tiles);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (m < M) v = ldg16(x + (size_t)m * row_bytes + (size_t)st * 64 + (lane >> 4) * 16);
    stg16(xt + p * 16, v);
  }
}

// D += A B as mma16 has it, in place.  Written as asm because the compiler, left to itself, gives the 16 x 16 instruction another
// register for its result than for its addend and copies accumulators around the loop (140 copies beside 192 matrix instructions).
// The operands are those of ordinary loads, which the compiler waits for; nothing but these instructions touches an accumulator
// between its first zero and the wait behind the loop.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gw_rsrc(const void *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}
template <typename T> __device__ __forceinline__ void gw_mma(f32x4 &d, const u32x4 &w, const u32x4 &x) {
  if constexpr (sizeof(T) == 2) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(w), "v"(x));
  } else {
    #pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(d) : "v"(w[j]), "v"(x[j]));
  }
}

// ---- epilogues of the wide kernel, straight from the accumulators (through a tile in LDS they took 9 to 19 thousand clocks of 80 to
// 270).  A wave's tile of 32 rows is two accumulators of 16 x 16 a block: lane (g, r16) holds activation rows r16 and 16 + r16 against
// weight rows g * 4 .. + 3.  Where a block pairs its rows (gate with up, a dimension with its RoPE partner, 8 rows further on: two
// lane groups) the upper half of one accumulator changes places with the lower half of the other: then lane (hh, gl, r16) holds row
// hh * 16 + r16 against weight rows gl * 4 .. + 3 in the first and 8 + gl * 4 .. + 3 in the second.
__device__ __forceinline__ void gw_pair(f32x4 &a, f32x4 &b) {
  #pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto s = __builtin_amdgcn_permlane32_swap(lane_bits(a[i]), lane_bits(b[i]), false, false);
    a[i] = lane_value<float>(s[0]);
    b[i] = lane_value<float>(s[1]);
  }
}
// 4 adjacent outputs of block 0 in y0 and of block 1 in y1 (lane gl holds outputs gl * 4 .. + 3 of the 8 of its row): afterwards lane gl
// holds the 8 outputs of block gl, 16 bytes of bf16.
__device__ __forceinline__ uint4 gw_join(const float (&y0)[4], const float (&y1)[4]) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  union { bf16x4 v; unsigned u[2]; } a, b;
  #pragma unroll
  for (int i = 0; i < 4; ++i) { a.v[i] = (bf16_t)y0[i]; b.v[i] = (bf16_t)y1[i]; }
  const auto p = __builtin_amdgcn_permlane16_swap(a.u[0], b.u[0], false, false), q = __builtin_amdgcn_permlane16_swap(a.u[1], b.u[1], false, false);
  return make_uint4(p[0], q[0], p[1], q[1]);
}

template <typename T, int EPI, int NP, int TW>
__global__ __launch_bounds__(64 * GW_W) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_gemm_wide(const GemmArgs a, int tiles, int mgroups, int m32_tiles, int gt) {
  extern __shared__ __align__(16) unsigned char gw_lds[];
  constexpr int NB = 2 * NP, STAGE = NB * GW_ST * 1024, XD = GW_ST;    // XD: steps in the ring of activations
  static_assert(GW_ST == GW_W, "a wave brings in one step of every block of a stage");
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  const int S = a.split_k;
  const int id = blockIdx.x, unit = (id / 8 / mgroups) * 8 + (id & 7), mgroup = (id / 8) % mgroups;
  if (unit >= tiles * S) return;                          // padding of the last group of 8 units (whole workgroup)
  const int tile = unit / S, split = unit % S;
  // the group's rows in sixteens, dealt to the waves one by one
  const int sub0 = mgroup * gt * 2, sub1 = min(sub0 + gt * 2, (a.M + 15) >> 4);
  auto sub_of = [&](int i) { return sub0 + wave + i * GW_W; };
  const int total_steps = a.Kd * (int)sizeof(T) / 64;
  const int ssh = __ffs(S) - 1;                           // S is 1, 2, 4 or 8
  const int s0 = (total_steps * split) >> ssh, s1 = (total_steps * (split + 1)) >> ssh;
  const int n = s1 - s0;
  const int P = (n + GW_ST - 1) / GW_ST;                   // stages
  const int nblk = gemm_blocks(EPI, a.seg_rows);

  // Loads go through buffer descriptors: per block (tile) a lane's offset that stays, and one scalar that moves along the reduction
  // axis (added up in vector registers for every load, the addresses took as many issue slots as the matrix instructions).  For the
  // weights it is a 32-bit offset (gemm_is_wide leaves a workgroup's weights of 4 GiB and more to the skinny kernel), for the activations,
  // of which there can be more, the descriptor's base.
  // Weights: this wave's step of every block of a stage, contiguous 1 KB pieces.  Lane l has piece l % 4 of row l / 4; in LDS a row's
  // pieces are permuted (piece g at g ^ (row / 4)), which leaves the fragment reads free of bank conflicts.  Blocks past the
  // end re-read the last one and are never stored, steps past the slice its last one and are never multiplied.
  const int blocks_here = min(NB, nblk - tile * NB);
  const auto w_rsrc = gw_rsrc((const unsigned char *)a.wt + (size_t)tile * NB * total_steps * 1024, (unsigned)blocks_here * total_steps * 1024u);
  const int wdst = wave * 1024 + (lane >> 2) * 64 + (((lane & 3) ^ (lane >> 4)) & 3) * 16;
  constexpr bool WO = NP < 6;                               // a block's offset in a vector register of its own, or (where these are scarce) a scalar one
  unsigned wo[NB];
  #pragma unroll
  for (int b = 0; b < NB; ++b) wo[b] = (unsigned)(min(b, blocks_here - 1) * total_steps) * 1024u + (WO ? lane * 16 : 0);
  u32x4 wr[NB];
  auto w_at = [&](int p) { return (unsigned)(s0 + min(p * GW_ST + wave, n - 1)) * 1024u; };
  auto load_w = [&](unsigned at, int b) { return WO ? __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, wo[b], at, 2) : __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane * 16, at + wo[b], 2); };   // non-temporal
  auto store_w = [&](int b, int slot, const u32x4 &w) { *reinterpret_cast<u32x4 *>(gw_lds + slot * STAGE + b * (GW_ST * 1024) + wdst) = w; };
  // Activations: sixteens past the end re-read the last one and are never stored, steps past the slice the last one
  const unsigned x_step = (unsigned)m32_tiles * 2048u;      // bytes of a step
  auto x_at = [&](int i) { return (const unsigned char *)a.xt + (size_t)(unsigned)(s0 + min(i, n - 1)) * x_step; };
  const int woff = r16 * 64 + ((g ^ (r16 >> 2)) & 3) * 16;
  u32x4 wf[2][NP];
  // fragment b of half-step j of the stage in slot u: half of the blocks against one step
  auto read_w = [&](int u, int j, int b) { return *reinterpret_cast<const u32x4 *>(gw_lds + woff + u * STAGE + ((j & 1) * NP + b) * (GW_ST * 1024) + (j >> 1) * 1024); };

  auto run = [&](auto tag) {                               // tag: sixteens of rows that this wave multiplies
    constexpr int NS = decltype(tag)::value;
    int xo[NS];
    #pragma unroll
    for (int i = 0; i < NS; ++i) xo[i] = min(sub_of(i), 2 * m32_tiles - 1) * 1024 + lane * 16;
    u32x4 xq[XD][NS];
    auto load_x = [&](const unsigned char *at, int i) { return __builtin_amdgcn_raw_buffer_load_b128(gw_rsrc(at, x_step), xo[i], 0, 0); };
    f32x4 acc[NB][NS];
    #pragma unroll
    for (int b = 0; b < NB; ++b)
      #pragma unroll
      for (int i = 0; i < NS; ++i) { acc[b][i] = (f32x4){0.f, 0.f, 0.f, 0.f}; asm volatile("" : "+a"(acc[b][i])); }
    {
      const unsigned w0 = w_at(0), w1 = w_at(1);
      #pragma unroll
      for (int b = 0; b < NB; ++b) wr[b] = load_w(w0, b);
      #pragma unroll
      for (int i = 0; i < XD - 1; ++i) {
        const unsigned char *at = x_at(i);
        #pragma unroll
        for (int t = 0; t < NS; ++t) xq[i][t] = load_x(at, t);
      }
      #pragma unroll
      for (int b = 0; b < NB; ++b) store_w(b, 0, wr[b]);
      #pragma unroll
      for (int b = 0; b < NB; ++b) wr[b] = load_w(w1, b);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    #pragma unroll
    for (int b = 0; b < NP; ++b) wf[0][b] = read_w(0, 0, b);
    constexpr int HSN = 2 * GW_ST, W0 = 1, WN = 4, WB = (NB + WN - 1) / WN;      // half-steps of a stage; the WN from W0 on write the next one
    const unsigned char *xp = nullptr;                     // where this half-step's loads of activations are from
    // jtag: half-step of stage p; utag: the stage's slot p % 2; whole: all the stage's steps are in the slice.  False: the slice has ended.
    auto half_step = [&](int p, unsigned wp, auto jtag, auto utag, auto whole) {
      constexpr int j = decltype(jtag)::value, u = decltype(utag)::value, MN = NP * NS;
      const int i = p * GW_ST + (j >> 1);
      if (!decltype(whole)::value && (j & 1) == 0 && i >= n) return false;  // (the same for every wave)
      if (j == HSN - 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the next stage is whole, this one read
      if ((j & 1) == 0) xp = x_at(i + XD - 1);           // into the registers of the step before
      // what else there is to do in this half-step, in order: the activations' loads, then every block's write and next load
      constexpr int nw = (j >= W0 && j - W0 < WN) ? (NB - (j - W0) * WB < WB ? NB - (j - W0) * WB : WB) : 0;
      constexpr int nx = (NS + 1 - (j & 1)) / 2, ops = nx + 2 * (nw > 0 ? nw : 0);
      auto op = [&](int k) {
        if (k < nx) { xq[((j >> 1) + XD - 1) % XD][2 * k + (j & 1)] = load_x(xp, 2 * k + (j & 1)); return; }
        const int b = (j - W0) * WB + (k - nx) / 2;
        if ((k - nx) % 2 == 0) store_w(b, u ^ 1, wr[b]); else wr[b] = load_w(wp, b);
      };
      auto read = [&](int b) { wf[(j + 1) & 1][b] = j < HSN - 1 ? read_w(u, j + 1, b) : read_w(u ^ 1, 0, b); };
      if (decltype(whole)::value) {
        // an LDS read ahead of every fragment's matrix instructions, the rest spread evenly between them
        #pragma unroll
        for (int b = 0; b < NP; ++b) {
          read(b);
          #pragma unroll
          for (int t = 0; t < NS; ++t) {
            gw_mma<T>(acc[(j & 1) * NP + b][t], wf[j & 1][b], xq[(j >> 1) % XD][t]);
            static_assert(ops <= 3 * MN, "at most three of them fall behind one instruction");
            const int m = b * NS + t, k = (m * ops + MN - 1) / MN;
            if (k * MN < (m + 1) * ops) op(k);
            if ((k + 1) * MN < (m + 1) * ops) op(k + 1);
            if ((k + 2) * MN < (m + 1) * ops) op(k + 2);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        #pragma unroll
        for (int b = 0; b < NP; ++b) read(b);
        #pragma unroll
        for (int k = 0; k < ops; ++k) op(k);
        #pragma unroll
        for (int b = 0; b < NP; ++b)
          #pragma unroll
          for (int t = 0; t < NS; ++t) gw_mma<T>(acc[(j & 1) * NP + b][t], wf[j & 1][b], xq[(j >> 1) % XD][t]);
        __builtin_amdgcn_sched_barrier(0);
      }
      return true;
    };
    auto stage = [&](int p, auto utag, auto whole) {
      const unsigned wp = w_at(p + 2);
      static_assert(HSN == 8, "the half-steps below");
      (void)(half_step(p, wp, GemmTag<0>{}, utag, whole) && half_step(p, wp, GemmTag<1>{}, utag, whole) &&
             half_step(p, wp, GemmTag<2>{}, utag, whole) && half_step(p, wp, GemmTag<3>{}, utag, whole) &&
             half_step(p, wp, GemmTag<4>{}, utag, whole) && half_step(p, wp, GemmTag<5>{}, utag, whole) &&
             half_step(p, wp, GemmTag<6>{}, utag, whole) && half_step(p, wp, GemmTag<7>{}, utag, whole));
    };
    int p = 0;
    for (; (p + 2) * GW_ST <= n; p += 2) {
      stage(p, GemmTag<0>{}, GemmTag<1>{});
      stage(p + 1, GemmTag<1>{}, GemmTag<1>{});
    }
    if (p < P) stage(p, GemmTag<0>{}, GemmTag<0>{});
    if (p + 1 < P) stage(p + 1, GemmTag<1>{}, GemmTag<0>{});
    // the last matrix instructions finish before anything else reads their accumulators (the compiler does not know what is in the asm)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    #pragma unroll
    for (int b = 0; b < NB; ++b)
      #pragma unroll
      for (int i = 0; i < NS; ++i) asm volatile("" : "+a"(acc[b][i]));

    const int gl = g & 1, hh = lane >> 5, b0 = tile * NB;    // b0: first row block of the workgroup
    #pragma unroll
    for (int t = 0; t < NS; t += 2) {
      if (sub_of(t) >= sub1) break;                          // (wave-uniform)
      // row of this lane where the two sixteens are paired (an odd last one with itself)
      const int m = sub_of(min(t + hh, NS - 1)) * 16 + r16;
      const bool row_ok = t + hh < NS && sub_of(t + hh) < sub1 && m < a.M;
      auto pair_of = [&](int b, f32x4 &lo, f32x4 &hi) { lo = acc[b][t]; hi = acc[b][min(t + 1, NS - 1)]; gw_pair(lo, hi); };
      if (EPI == EPI_ARGMAX) {
        // Which columns of a ragged last tile exist is asked anew for every tile of rows: shared by them, the answers were 16 NP
        // lane masks (up to 200 scalar registers spilled).
        #pragma unroll
        for (int c = 0; c < 2 && t + c < NS; ++c) {
          float bv = -__builtin_huge_valf(); int bi = 0x7fffffff;
          // Columns in descending order: at equal values the lower one comes later
          const int n0 = b0 * 16 + g * 4;
          int live = a.seg_rows - n0;
          asm volatile("" : "+v"(live));
          #pragma unroll
          for (int b = NB - 1; b >= 0; --b) {
            #pragma unroll
            for (int i = 3; i >= 0; --i) {
              const float v = acc[b][t + c][i];
              if (b * 16 + i < live && v >= bv) { bv = v; bi = n0 + b * 16 + i; }
            }
            if (b % 2 == 0) __builtin_amdgcn_sched_barrier(0);
          }
          best_of_groups(bv, bi);
          const int mg = sub_of(t + c) * 16 + r16;
          if (g == 0 && sub_of(t + c) < sub1 && mg < a.M) {
            a.amax_val[(size_t)tile * a.M + mg] = bv;
            a.amax_idx[(size_t)tile * a.M + mg] = bi;
          }
        }
      }
      if (EPI == EPI_STORE || (EPI == EPI_ARGMAX && a.logits)) {
        // [split_k][M][N] partial sums (one slab of them: the logits): 4 adjacent columns a lane, one by one in a ragged last tile
        // and in a caller's logits that begin anywhere
        const int N = a.seg_rows;
        float *slab = EPI == EPI_STORE ? a.out + (size_t)split * a.M * N : a.logits;
        const bool pieces = (N & 3) == 0 && ((uintptr_t)slab & 15) == 0;
        #pragma unroll
        for (int c = 0; c < 2 && t + c < NS; ++c) {
          const int mg = sub_of(t + c) * 16 + r16;
          if (sub_of(t + c) >= sub1 || mg >= a.M) continue;
          float *dst = slab + (size_t)mg * N + b0 * 16 + g * 4;
          const int left = N - (b0 * 16 + g * 4);
          #pragma unroll
          for (int b = 0; b < NB; ++b) {
            const f32x4 v = acc[b][t + c];
            if (pieces && left - b * 16 >= 4) {
              *reinterpret_cast<f32x4 *>(dst + b * 16) = v;
            } else {
              #pragma unroll
              for (int i = 0; i < 4; ++i)
                if (b * 16 + i < left) dst[b * 16 + i] = v[i];
            }
          }
        }
      }
      if (EPI == EPI_SWIGLU) {
        const int f = a.seg_rows;
        T *act = (T *)a.act;
        #pragma unroll
        for (int pr = 0; pr < NP; ++pr) {
          float y[2][4];
          #pragma unroll
          for (int e = 0; e < 2; ++e) {
            f32x4 gate, up;
            pair_of(2 * pr + e, gate, up);
            #pragma unroll
            for (int i = 0; i < 4; ++i) y[e][i] = silu_f(gate[i]) * up[i];
          }
          if constexpr (sizeof(T) == 2) {
            const uint4 v = gw_join(y[0], y[1]);
            const int j0 = (b0 + 2 * pr + gl) * 8;
            if (!row_ok || j0 >= f) continue;
            T *dst = act + (size_t)m * f + j0;
            if (a.act_tiles) {                               // tiled for the wide GEMM that follows (f is a multiple of 16)
              stg16(act + xt_index<T>(m, j0, a.act_tiles), v);
            } else if (j0 + 8 <= f && (f & 3) == 0) {
              *reinterpret_cast<uint2 *>(dst) = make_uint2(v.x, v.y);
              *reinterpret_cast<uint2 *>(dst + 4) = make_uint2(v.z, v.w);
            } else {
              const unsigned w4[4] = {v.x, v.y, v.z, v.w};
              #pragma unroll
              for (int i = 0; i < 8; ++i)
                if (j0 + i < f) reinterpret_cast<unsigned short *>(dst)[i] = (unsigned short)(w4[i / 2] >> (16 * (i & 1)));
            }
          } else {
            #pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int j0 = (b0 + 2 * pr + e) * 8 + gl * 4;
              if (!row_ok || j0 >= f) continue;
              if (a.act_tiles) store4<T>(act + xt_index<T>(m, j0, a.act_tiles), y[e]);
              else if (j0 + 4 <= f && (f & 3) == 0) store4<T>(act + (size_t)m * f + j0, y[e]);
              else
                for (int i = 0; i < 4 && j0 + i < f; ++i) act[(size_t)m * f + j0 + i] = Elem<T>::from_f32(y[e][i]);
            }
          }
        }
      }
      if (EPI == EPI_QKV_ROPE) {
        // d_h is a power of two (checked at launch): heads and dims come from shifts.  What a lane needs from global memory
        // (32 bytes of the cos/sin table a block) is requested QB blocks ahead of the stores.
        constexpr int QB = NB % 4 ? 2 : 4, PIECE = 64 / (int)sizeof(T);
        const int d_h = a.d_h, d = a.n_heads * d_h, bps = d >> 4, bph = d_h >> 4, bsh = __ffs(bph) - 1, half = d_h >> 1;
        const int bb = row_ok ? m / a.T_nodes : 0, node = row_ok ? m - bb * a.T_nodes : 0, L = a.kv_len[bb];
        const bool kv_ok = row_ok && L >= 0 && L + a.T_nodes <= a.max_kv;
        if (row_ok && !kv_ok && node == 0) atomicOr(a.dev_status, 2u);
        const size_t cache = (size_t)a.max_kv * d_h;
        T *q_row = (T *)a.q_out + (size_t)(row_ok ? m : 0) * d, *kb = (T *)a.k_cache + (size_t)bb * a.n_heads * cache, *vb = (T *)a.v_cache + (size_t)bb * a.n_heads * cache;
        const size_t v_at = v_tiled_index<T>(kv_ok ? L + node : 0, 0, d_h);
        const float2 *cs_row = a.rope_cs + (size_t)(row_ok ? m : 0) * half + gl * 4;
        auto seg_of = [&](int b) { return (b >= 2 * bps) ? 2 : (b >= bps) ? 1 : 0; };
        float4 tab[2][QB][2];
        auto load_tab = [&](int q, float4 (&tb)[QB][2]) {
          #pragma unroll
          for (int k = 0; k < QB; ++k) {
            const int b = min(b0 + q * QB + k, nblk - 1), bl = b - seg_of(b) * bps;
            const float4 *p = reinterpret_cast<const float4 *>(cs_row + (bl & (bph - 1)) * 8);
            tb[k][0] = p[0]; tb[k][1] = p[1];
          }
        };
        load_tab(0, tab[0]);
        #pragma unroll
        for (int q = 0; q < NB / QB; ++q) {
          if (q + 1 < NB / QB) load_tab(q + 1, tab[(q + 1) & 1]);
          #pragma unroll
          for (int k = 0; k < QB; k += 2) {
            const int lb = q * QB + k, b = b0 + lb;
            if (b >= nblk) continue;
            float y[2][2][4];                                // [block][dims, partners]
            #pragma unroll
            for (int e = 0; e < 2; ++e) {
              f32x4 lo, hi;
              pair_of(lb + e, lo, hi);
              const float4 c0 = tab[q & 1][k + e][0], c1 = tab[q & 1][k + e][1];
              const float cs[4] = {c0.x, c0.z, c1.x, c1.z}, sn[4] = {c0.y, c0.w, c1.y, c1.w};
              const bool rot = seg_of(b + e) < 2;            // (uniform)
              #pragma unroll
              for (int i = 0; i < 4; ++i) {
                float y1, y2;
                rope_pair(lo[i], hi[i], cs[i], sn[i], y1, y2);
                y[e][0][i] = rot ? y1 : lo[i];
                y[e][1][i] = rot ? y2 : hi[i];
              }
            }
            // where 8 outputs from block bl's dim e0 on go (q and k): e0 and e0 + d_h / 2
            auto dst_of = [&](int seg, int bl, int e0, T *&d1, T *&d2) {
              const int head = bl >> bsh;
              if (seg == 0) { d1 = q_row + head * d_h + e0; d2 = d1 + half; }
              else { T *kc = kb + (size_t)head * cache; d1 = kc + k_tiled_index<T>(L + node, e0, d_h); d2 = kc + k_tiled_index<T>(L + node, e0 + half, d_h); }
            };
            const int s0_ = seg_of(b), s1_ = seg_of(b + 1);
            if (sizeof(T) == 2 && s0_ == s1_ && s0_ < 2 && b + 1 < nblk) {
              const uint4 v1 = gw_join(y[0][0], y[1][0]), v2 = gw_join(y[0][1], y[1][1]);
              const int bl = b + gl - s0_ * bps;
              T *d1, *d2;
              dst_of(s0_, bl, (bl & (bph - 1)) * 8, d1, d2);
              if (s0_ == 0 ? row_ok : kv_ok) { stg16(d1, v1); stg16(d2, v2); }
              continue;
            }
            #pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int seg = e ? s1_ : s0_, bl = b + e - seg * bps;
              if (b + e >= nblk) continue;
              if (seg == 2) {
                if (!kv_ok) continue;
                T *dst = vb + (size_t)(bl >> bsh) * cache + v_at + ((bl & (bph - 1)) * 16 + gl * 4) * PIECE;
                #pragma unroll
                for (int i = 0; i < 4; ++i) { dst[i * PIECE] = Elem<T>::from_f32(y[e][0][i]); dst[(8 + i) * PIECE] = Elem<T>::from_f32(y[e][1][i]); }
              } else {
                T *d1, *d2;
                dst_of(seg, bl, (bl & (bph - 1)) * 8 + gl * 4, d1, d2);
                if (seg == 0 ? row_ok : kv_ok) { store4<T>(d1, y[e][0]); store4<T>(d2, y[e][1]); }
              }
            }
          }
        }
      }
    }
  };
  const int mine = (sub1 - sub0 - wave + GW_W - 1) / GW_W;   // (what a wave multiplies beyond its own is never stored)
  if (mine >= 2 * TW) run(GemmTag<2 * TW>{});
  else if (TW == 1 || mine == 2 * TW - 1) run(GemmTag<2 * TW - 1>{});
  else run(GemmTag<(TW > 1 ? 2 * TW - 2 : 1)>{});
}

// Row-major -> tiled (see the layout above).  One thread per 16-byte piece of the tiled buffer.
template <typename T, int EPI>
__global__ __launch_bounds__(256) void k_pack_weights(const GemmArgs a, unsigned char *dst) {
  const int total_steps = a.Kd * (int)sizeof(T) / 64;
  const size_t pieces = (size_t)gemm_blocks(EPI, a.seg_rows) * total_steps * 64;   // 64 pieces of 16 bytes per fragment
  for (size_t p = (size_t)blockIdx.x * 256 + threadIdx.x; p < pieces; p += (size_t)gridDim.x * 256) {
    const int g = (int)(p & 3), r16 = (int)((p >> 2) & 15);
    const size_t frag = p >> 6;
    const int st = (int)(frag % total_steps);
    const int blk = (int)(frag / total_steps);
    const RowMap rm = map_block<EPI>(a, blk, r16);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (rm.valid) {
      const void *wm = (rm.seg == 0) ? a.w0 : (rm.seg == 1) ? a.w1 : a.w2;
      v = ldg16((const unsigned char *)wm + ((size_t)rm.n * a.Kd * sizeof(T) + (size_t)st * 64 + g * 16));
    }
    stg16(dst + p * 16, v);
  }
}

size_t gemm_tiled_bytes(int epi, int seg_rows, int Kd, int elem_bytes) {
  return (size_t)gemm_blocks(epi, seg_rows) * 16 * (size_t)Kd * elem_bytes;
}

template <typename T>
hipError_t launch_pack_weights(hipStream_t st, int epi, const GemmArgs &a, void *dst) {
  if (a.Kd < 1 || (a.Kd * (int)sizeof(T)) % 64) return hipErrorInvalidValue;
  if (epi == EPI_QKV_ROPE && (a.d_h % 16 || a.seg_rows != a.n_heads * a.d_h)) return hipErrorInvalidValue;
  const size_t pieces = gemm_tiled_bytes(epi, a.seg_rows, a.Kd, (int)sizeof(T)) / 16;
  const int blocks = (int)std::min<size_t>((pieces + 255) / 256, 65536);
  unsigned char *d8 = (unsigned char *)dst;
  switch (epi) {
    case EPI_STORE: hipLaunchKernelGGL((k_pack_weights<T, EPI_STORE>), dim3(blocks), dim3(256), 0, st, a, d8); break;
    case EPI_QKV_ROPE: hipLaunchKernelGGL((k_pack_weights<T, EPI_QKV_ROPE>), dim3(blocks), dim3(256), 0, st, a, d8); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((k_pack_weights<T, EPI_SWIGLU>), dim3(blocks), dim3(256), 0, st, a, d8); break;
    case EPI_ARGMAX: hipLaunchKernelGGL((k_pack_weights<T, EPI_ARGMAX>), dim3(blocks), dim3(256), 0, st, a, d8); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template hipError_t launch_pack_weights<float>(hipStream_t, int, const GemmArgs &, void *);
template hipError_t launch_pack_weights<bf16_t>(hipStream_t, int, const GemmArgs &, void *);

// tgt[m] = index of the best of the per-tile winners (ties -> lower index); one wave per row
__global__ __launch_bounds__(64) void k_argmax_fold(const float *amax_val, const int32_t *amax_idx, int tiles, int M,
                                                    int32_t *tgt) {
  const int mg = blockIdx.x, lane = threadIdx.x;
  float bv = -__builtin_huge_valf(); int bi = 0x7fffffff;
  for (int t = lane; t < tiles; t += WAVE) {
    const float v = amax_val[(size_t)t * M + mg];
    const int i = amax_idx[(size_t)t * M + mg];
    if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
  }
  wave_best(bv, bi);
  if (lane == 0) tgt[mg] = bi;
}

// out[i] = sum_s slabs[s][i], s ascending
__global__ __launch_bounds__(256) void k_sum_slabs(const float *slabs, int S, size_t n, float *out) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    float v = slabs[i];
    for (int s = 1; s < S; ++s) v += slabs[(size_t)s * n + i];
    out[i] = v;
  }
}

hipError_t launch_sum_slabs(hipStream_t st, const float *slabs, int S, size_t n, float *out) {
  int blocks = (int)((n + 255) / 256);
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(k_sum_slabs, dim3(blocks), dim3(256), 0, st, slabs, S, n, out);
  return hipGetLastError();
}

hipError_t launch_argmax_fold(hipStream_t st, const float *amax_val, const int32_t *amax_idx, int tiles, int M,
                              int32_t *tgt) {
  hipLaunchKernelGGL(k_argmax_fold, dim3(M), dim3(64), 0, st, amax_val, amax_idx, tiles, M, tgt);
  return hipGetLastError();
}

// Tile height and reduction split of the skinny kernel for one GEMM.  Model, in units of one weight fragment: a workgroup's
// time is its steps times (nb fragments + 2 for its share of the activation chunk); the kernel's time
// is that times the number of rounds the grid needs on 256 CUs; every split beyond the first costs the
// write and the later read of one more float32 slab.  The two constants are fitted to measurements of
// the 7B shapes (Wo: 4 blocks x 4 splits beats 2 x 2 and 8 x 8; down: 4 x 4 beats 8 x 8).
static GemmPlan plan_skinny(int epi, int seg_rows, int Kd, int elem_bytes, int M, int split_req) {
  GemmPlan best{};
  const int blocks = gemm_blocks(epi, seg_rows);
  const int total_steps = Kd * elem_bytes / 64;
  const int mblocks = (M + GM_BM - 1) / GM_BM;
  const bool fused = epi != EPI_STORE;
  const double slab_units = fused ? 0.0 : (double)M * seg_rows * 1.0e-4 + 2.0;   // per extra split
  double best_cost = 1e300;
  best.blocks = blocks;
  best.mgroups = mblocks;
  for (int s = 1; s <= 8; s *= 2) {
    if (split_req > 0 && s != split_req) continue;
    if (split_req == 0 && (fused ? s > 1 : (s > 1 && total_steps / s < 2 * GM_STEPS))) continue;
    for (int nb = GM_MIN_NB; nb <= GM_MAX_NB; ++nb) {
      if (nb > std::max(blocks, GM_MIN_NB)) break;
      const int tiles = (blocks + nb - 1) / nb;
      const long wgs = (long)tiles * s * mblocks;
      const long rounds = (wgs + 255) / 256;
      const double cost = (double)rounds * ((total_steps + s - 1) / s) * (nb + 2) + slab_units * (s - 1);
      if (cost <= best_cost) { best_cost = cost; best.nb = nb; best.split = s; best.tiles = tiles; }
    }
  }
  return best;
}

// The wide kernel's tiles for a given split: groups of gt tiles of 32 activation rows (up to six sixteens a wave) against nb weight row
// blocks.  The price is in us.  A step of 64 bytes of k takes what lasts longer: the matrix instructions of the busiest wave and the
// fragments that it reads from LDS for them, at a clock that is lower the fuller the chip and the busier the other waves (in bf16, where the power
// sets it); or what the workgroup takes in, 2 KB for every tile, from further away the more rows there are, and 1 KB for every block (of which
// the groups share the way from HBM), faster on a chip that is not full.  A part of the shorter one does not hide behind it.  A compute
// unit has one workgroup at a time, and the workgroups are dealt to the XCDs in eights: 252 of them in three groups can mean 33 on one
// XCD and a second round (6656 x 17920 over 320 rows: 172 us against 106).
// Fitted to 21,916 measurements of launches in a row (bf16 at 7B, 13B and 33B widths and 2048 over 80 to 768 rows, at nine widths from 512
// to 8192 over 65 to 128, at four over 208 to 8192; float32 at five widths from 256 to 4096 over 144 to 768): 6 % deviation.  Over the shapes the
// picks take 39.42 ms where the best plans take 39.18 (80 to 768 rows), 9.66 where 9.62 (65 to 128), 24.07 where 24.00 (208 to 8192), and
// 39.73 where 39.69 (float32).  (The price of the 32 x 32 form took 39.62, 9.67, 24.14 and 41.75.)
static GemmPlan plan_wide(int epi, int seg_rows, int Kd, int elem_bytes, int M, int split) {
  GemmPlan best{};
  const int blocks = gemm_blocks(epi, seg_rows);
  const int steps = (Kd * elem_bytes / 64 + split - 1) / split;
  best.blocks = blocks;
  best.wide = true;
  best.split = split;
  best.cost = 1e300;
  const int mt = (M + 31) / 32, most = GW_W * (elem_bytes == 4 ? 2 : GW_MAX_TW);
  for (int mg = (mt + most - 1) / most; mg <= (mt + 2) / 3; ++mg) {   // (three tiles or more a group)
    const int gt = (mt + mg - 1) / mg, tw = (gt + GW_W - 1) / GW_W;
    if ((mg - 1) * gt >= mt) continue;                                // fewer groups of as many tiles do
    const int ns = (std::min(2 * gt, (M + 15) / 16) + GW_W - 1) / GW_W;   // sixteens of the busiest wave
    for (int np = 2; np <= GW_MAX_NP; ++np) {
      if (!gw_built(elem_bytes, np, tw)) continue;
      const int nb = 2 * np, tiles = (blocks + nb - 1) / nb;
      const long on_xcd = (long)((tiles * split + 7) / 8) * mg, rounds = (on_xcd + 31) / 32;
      const double full = (double)on_xcd / (32.0 * rounds);
      const double mma = elem_bytes == 4 ? nb * (0.0472 * ns + 0.0034) : nb * (0.0037 * ns + 0.0034) * (1.0 + full * (0.748 * gt / ns - 0.576));
      const double intake = (0.0151 * gt * (1.0 + 0.0037 * mt) + 0.0215 * nb * (0.43 + 0.57 / mg)) * (0.65 + 0.35 * full);
      const double step = std::max(mma, intake) + 0.309 * std::min(mma, intake) + 0.052;
      const double cost = (double)rounds * (steps * step + 0.585 + 0.213 * nb * ns) + 1.91;
      if (cost < best.cost) { best.cost = cost; best.nb = nb; best.tiles = tiles; best.mgroups = mg; best.tw = tw; best.gt = gt; }
    }
  }
  return best;
}

// Slabs that the reduction axis of a matrix is cut into.  The one choice of a plan that the result depends on: inside a
// slab both kernels add the same products in the same order, so their bits are the same.  Therefore it is a rule on the shape
// alone.  Up to 128 rows it is the skinny kernel's, for whichever kernel runs and however the weights are stored: tiled and
// row-major weights give the same bits there.  Beyond (tiled weights), the count whose plan is priced lowest with 0.6 us a further slab and 0.9
// for every million of its outputs (its way out of the kernel and into the next one).
// Measured with the fold behind the launch, W_o and W_down over 129 to 768 rows, ms of all shapes of a size with these picks / with the
// best: bf16 from 512 x 512 to 1 Mi weights 0.22 / 0.20, to 4 Mi 0.40 / 0.38, to 16 Mi 1.20 / 1.18, beyond (to 6656 x 17920) 4.36 / 4.33;
// float32 from 256 x 256 0.58 / 0.58, 0.47 / 0.47, 1.09 / 1.08, 3.37 / 3.34.
static int gemm_split(int epi, int seg_rows, int Kd, int elem_bytes, int M, bool tiled) {
  if (epi != EPI_STORE) return 1;                           // fused epilogues need complete sums
  if (!tiled || M <= 2 * GM_BM) return plan_skinny(epi, seg_rows, Kd, elem_bytes, M, 0).split;
  const int steps = Kd * elem_bytes / 64;
  double best_cost = 1e300;
  int best = 1;
  for (int s = 1; s <= 8 && (s == 1 || steps / s >= 16); s *= 2) {
    const double cost = plan_wide(epi, seg_rows, Kd, elem_bytes, M, s).cost + (0.9e-6 * M * seg_rows + 0.6) * (s - 1);
    if (cost < best_cost) { best_cost = cost; best = s; }
  }
  return best;
}

// Which kernel.  Up to 64 rows the skinny one, from 129 on the wide one.  In between (two blocks of 64 rows, or three and
// four tiles of 32) mostly the wide one; the skinny kernel still does better where the matrix is small, or one round of its
// workgroups with a split axis (us, skinny / wide, 128 rows: QKV 2048 wide 13.6 / 14.4, 3072 21.6 / 22.7, W_o 4096 x 4096 13.6 / 14.3,
// 5120 x 5120 18.0 / 19.7; but W_down 4096 x 11008 29.0 / 25.2, gate/up 2 x 11008 x 4096 44 / 38, QKV 5120 wide 46 / 40, the head
// 32000 x 4096 73 / 48).  Prices in us for equal slabs; over 315 shapes at nine widths from 512 to 8192 and 65 to 128 rows: always the
// wide kernel takes 9659 us over all of them, always the skinny one 12837, this rule 9585, the better choice each time 9572.
// float32 keeps to the skinny kernel, whose sums row-major weights have.
bool gemm_is_wide(int epi, int seg_rows, int Kd, int elem_bytes, int M, bool tiled) {
  const int mblocks = (M + GM_BM - 1) / GM_BM;
  if (!tiled || mblocks < 2 || (long long)Kd * elem_bytes / 64 * (2 * GW_MAX_NP * 1024) > 0xffffffffLL) return false;   // (offsets in a workgroup's weights have 32 bits)
  if (mblocks > 2) return true;
  if (elem_bytes == 4) return false;
  const int split = gemm_split(epi, seg_rows, Kd, elem_bytes, M, tiled);
  const GemmPlan s = plan_skinny(epi, seg_rows, Kd, elem_bytes, M, split), w = plan_wide(epi, seg_rows, Kd, elem_bytes, M, split);
  const double steps = (double)(Kd * elem_bytes / 64) / split;
  const double us_s = (double)(((long)s.tiles * split * mblocks + 255) / 256) * (2.4 + steps * (0.0273 * s.nb + 0.0446)) + 2.27;
  return w.cost + 1.2 < us_s;
}

GemmPlan gemm_plan(int epi, int seg_rows, int Kd, int elem_bytes, int M, int split_req, bool tiled) {
  const int split = split_req > 0 ? split_req : gemm_split(epi, seg_rows, Kd, elem_bytes, M, tiled);
  return gemm_is_wide(epi, seg_rows, Kd, elem_bytes, M, tiled) ? plan_wide(epi, seg_rows, Kd, elem_bytes, M, split)
                                                               : plan_skinny(epi, seg_rows, Kd, elem_bytes, M, split);
}

size_t gemm_xt_bytes(int M, int Kd, int elem_bytes) { return (size_t)((M + 31) / 32) * 32 * (size_t)Kd * elem_bytes; }

template <typename T, int EPI, int NP, int TW>
static hipError_t launch_wide_np(hipStream_t st, const GemmArgs &a, const GemmPlan &pl, int m32_tiles, dim3 grid, hipEvent_t ev_start, hipEvent_t ev_stop) {
  constexpr size_t smem = (size_t)2 * 2 * NP * GW_ST * 1024;            // two stages of weights
  static_assert(smem <= 160 * 1024, "LDS of one workgroup");
  const dim3 block(64 * GW_W);
  static bool attr_set = false;                           // once per instantiation and process
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)k_gemm_wide<T, EPI, NP, TW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (ev_start && ev_stop)
    hipExtLaunchKernelGGL((k_gemm_wide<T, EPI, NP, TW>), grid, block, smem, st, ev_start, ev_stop, 0, a, pl.tiles, pl.mgroups, m32_tiles, pl.gt);
  else
    hipLaunchKernelGGL((k_gemm_wide<T, EPI, NP, TW>), grid, block, smem, st, a, pl.tiles, pl.mgroups, m32_tiles, pl.gt);
  return hipGetLastError();
}

template <typename T, int EPI>
static hipError_t launch_wide(hipStream_t st, const GemmArgs &a, const GemmPlan &pl, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (!a.wt || !a.xt || pl.gt < 1 || pl.tw != (pl.gt + GW_W - 1) / GW_W) return hipErrorInvalidValue;
  const int m32_tiles = (a.M + 31) / 32, row_bytes = a.Kd * (int)sizeof(T);
  if ((long long)pl.mgroups * pl.gt < m32_tiles) return hipErrorInvalidValue;   // groups cover every row
  const size_t pieces = (size_t)(row_bytes / 64) * m32_tiles * 128;
  GemmArgs aw = a;
  if (a.x_tiled) aw.xt = const_cast<void *>(a.x);         // the producer of x wrote it tiled
  else hipLaunchKernelGGL((k_tile_rows<T>), dim3((unsigned)std::min<size_t>((pieces + 255) / 256, 4096)), dim3(256), 0, st,
                          (const unsigned char *)a.x, a.M, row_bytes, m32_tiles, (unsigned char *)a.xt);
  const long long wgs = (long long)((pl.tiles * a.split_k + 7) / 8) * pl.mgroups * 8;
  if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs);
  #define GW_LAUNCH(NP_, TW_)                                                                                   \
    if constexpr (gw_built((int)sizeof(T), NP_, TW_))                                                            \
      if (pl.nb == 2 * NP_ && pl.tw == TW_) return launch_wide_np<T, EPI, NP_, TW_>(st, aw, pl, m32_tiles, grid, ev_start, ev_stop)
  GW_LAUNCH(2, 1); GW_LAUNCH(3, 1); GW_LAUNCH(4, 1); GW_LAUNCH(5, 1);
  GW_LAUNCH(2, 2); GW_LAUNCH(3, 2); GW_LAUNCH(4, 2); GW_LAUNCH(5, 2); GW_LAUNCH(6, 2); GW_LAUNCH(8, 2);
  GW_LAUNCH(2, 3); GW_LAUNCH(3, 3); GW_LAUNCH(4, 3); GW_LAUNCH(5, 3);
  #undef GW_LAUNCH
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_gemm(hipStream_t st, int epi, const GemmArgs &a_in, hipEvent_t ev_start, hipEvent_t ev_stop) {
  GemmArgs a = a_in;
  if (a.M < 1 || a.Kd < 1 || (a.Kd * (int)sizeof(T)) % 64) return hipErrorInvalidValue;
  if (a.split_k != 1 && a.split_k != 2 && a.split_k != 4 && a.split_k != 8) return hipErrorInvalidValue;
  if (epi != EPI_STORE && a.split_k != 1) return hipErrorInvalidValue;     // fused epilogues need complete sums
  if (epi == EPI_QKV_ROPE && (a.d_h < 16 || (a.d_h & (a.d_h - 1)) || a.seg_rows != a.n_heads * a.d_h || !a.rope_cs)) return hipErrorInvalidValue;
  const GemmPlan pl = gemm_plan(epi, a.seg_rows, a.Kd, (int)sizeof(T), a.M, a.split_k, a.wt != nullptr && a.xt != nullptr);
  a.nb = pl.nb;
  if (!pl.wide && (a.x_tiled || a.act_tiles)) return hipErrorInvalidValue;   // only the wide kernel knows the tiled activations
  if (pl.wide) {
    switch (epi) {
      case EPI_STORE: return launch_wide<T, EPI_STORE>(st, a, pl, ev_start, ev_stop);
      case EPI_QKV_ROPE: return launch_wide<T, EPI_QKV_ROPE>(st, a, pl, ev_start, ev_stop);
      case EPI_SWIGLU: return launch_wide<T, EPI_SWIGLU>(st, a, pl, ev_start, ev_stop);
      case EPI_ARGMAX: return launch_wide<T, EPI_ARGMAX>(st, a, pl, ev_start, ev_stop);
      default: return hipErrorInvalidValue;
    }
  }
  const int tiles = pl.tiles;
  const int mblocks = (a.M + GM_BM - 1) / GM_BM;
  const long long wgs = (long long)((tiles * a.split_k + 7) / 8) * mblocks * 8;     // see the index mapping in the kernel
  if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs), block(64 * (a.nb + GM_NLW));
  // With a pair of events the launch itself carries them: they take the kernel's own begin and end time stamps,
  // so reading them costs the stream nothing and includes nothing but the kernel.
  #define GM_LAUNCH(E)                                                                                           \
    if (ev_start && ev_stop) {                                                                                   \
      if (a.wt) hipExtLaunchKernelGGL((k_gemm_skinny<T, E, true>), grid, block, 0, st, ev_start, ev_stop, 0, a, tiles);  \
      else hipExtLaunchKernelGGL((k_gemm_skinny<T, E, false>), grid, block, 0, st, ev_start, ev_stop, 0, a, tiles);      \
    } else if (a.wt) hipLaunchKernelGGL((k_gemm_skinny<T, E, true>), grid, block, 0, st, a, tiles);              \
    else hipLaunchKernelGGL((k_gemm_skinny<T, E, false>), grid, block, 0, st, a, tiles)
  switch (epi) {
    case EPI_STORE: GM_LAUNCH(EPI_STORE); break;
    case EPI_QKV_ROPE: GM_LAUNCH(EPI_QKV_ROPE); break;
    case EPI_SWIGLU: GM_LAUNCH(EPI_SWIGLU); break;
    case EPI_ARGMAX: GM_LAUNCH(EPI_ARGMAX); break;
    default: return hipErrorInvalidValue;
  }
  #undef GM_LAUNCH
  return hipGetLastError();
}
template hipError_t launch_gemm<float>(hipStream_t, int, const GemmArgs &, hipEvent_t, hipEvent_t);
template hipError_t launch_gemm<bf16_t>(hipStream_t, int, const GemmArgs &, hipEvent_t, hipEvent_t);

}  // namespace amph

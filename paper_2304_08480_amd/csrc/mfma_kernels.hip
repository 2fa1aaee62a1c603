// bf16 MFMA path ("materialized"): the two b x B logit blocks are computed once on the matrix cores,
// their un-normalised softmax numerators are kept in bf16, and the two gradient contractions of each
// block (Eq. 4-6) are MFMA GEMMs over those numerators.  12*b*B*d executed flops per call.
//
// For one block with query rows X (b x d, the rank's rows) and key rows Y (B x d):
//   z_ij   = s <x_i, y_j>                      z2 = z * log2(e)   (all exponentials are base 2)
//   ref2_i = z2 of the positive pair (i, label_i), lifted where needed so that no key of the positive's norm gives a
//            z2_ij - ref2_i above 100 (overflow guard, Cauchy-Schwarz)
//   E_ij   = exp2(z2_ij - ref2_i)  for j != label_i, stored as bf16 (b x B);  E_i,label = 0 in the
//            store and kept separately in fp32 as e_i
//   tot_i  = sum_j E_ij + e_i,  beta_i = 1/tot_i,  P_ij = beta_i E_ij,
//   ce_i   = log(tot_i / e_i),  P_i,label - 1 = -(sum_j E_ij)/tot_i       (no cancellation)
//   query-side gradient  gX_i = c s [ beta_i (E Y)_i + (P_i,label - 1) y_label ]
//   key-side gradient    gY_j = c s [ sum_i E_ij beta_i x_i  (+ (P_i,label - 1) x_i  if j = label_i) ]
//   d/ds share           c <gX_i / (c s), x_i>  summed over i   (sum_ij G_ij S_ij = <G Y, X>)
// Since lse_i >= z_i,label, every E_ij that underflows is negligible against the row total.  Where the guard lifts ref2_i so
// far above every logit of the row that its total falls below 2^-60 (rows of large norm whose cosines are all small), or
// keys of much larger norm than the positive's take a numerator above 2^101, k_row_merge redoes the row's group of 64 with
// the true row maxima as references (a slow path for inputs that are not CLIP-like).
//
// One NT tile main loop (mfma_tile.h: 256x256x64 by 8 waves, or 128x128x64 by 4, of MFMA 16x16x32 blocks, operands
// loaded global -> LDS directly into a ring of five units) serves all three contractions; operands whose
// reduction index is not the contiguous one in memory are read from LDS with transposing loads.
#include "common.h"
#include "mfma_tile.h"

namespace disco {
namespace {

using namespace tile;

constexpr float LOG2E = 1.4426950408889634f;
constexpr float REF_HEADROOM = 100.f;                    // largest exponent (base 2) a stored numerator should reach
// A row whose total lies below the floor has lost terms.  One with a partial sum over a tile's keys above the limit may hold
// numerators the guard does not allow (keys of the positive's norm reach it only if two of a tile are copies of the query and
// the positive is nowhere near it): times a key of large features they leave fp32, and 1 / total times a short row's leave bf16.
constexpr float ROW_TOTAL_FLOOR = 0x1p-60f, ROW_PART_MAX = 0x1p101f;

constexpr int BM = 256, BN = 256, NTHREADS = Cfg<256>::NTHREADS;     // the symmetric path's tiles

// The tile kernels come in two sizes, T = 256 (one workgroup of 8 waves per compute unit) and T = 128 (4 waves, two
// workgroups per compute unit); make_plan chooses.
template <int T>
constexpr int LOGIT_SMEM_BYTES = Cfg<T>::SMEM_BYTES;
template <int T>
constexpr int GEMM_SMEM_BYTES = OUT_SMEM_BYTES<T> > Cfg<T>::SMEM_BYTES ? OUT_SMEM_BYTES<T> : Cfg<T>::SMEM_BYTES;

// ------------------------------------------------------------------------------------------------
struct BlockPtrs {
  const uint16_t* X;     // b x d, the rank's rows
  const uint16_t* Y;     // B x d
  uint16_t* E;           // b x W stored numerators of one key panel, in 16-byte atoms (e_index)
  float* lpart;          // (2B/T) x b partial row sums (label column excluded) of logit tiles of size T
  float* ediag;          // b: numerator of the label column
  float* zd2;            // b: z2 of the positive pair
  float* ref2;           // b: exponent reference of the row
  float* beta;           // b
  float* gdiag;          // b: P_label - 1
  float* ce;             // b
  float* rowds;          // b
  uint16_t* Xs;          // d x b: (beta_i x_i)^T in bf16
  float* part;           // splitK x b x d partial query-side products
  float* kpart;          // key_splits x B x d partial key-side products (only where the plan splits that reduction)
  float* gq;             // query-side gradient destination (gI for block A, gT for block C), B x d
  float* gk;             // key-side gradient destination, B x d
};
struct Blocks {
  BlockPtrs z[2];
  int variant;           // LOSS_CLIP or LOSS_NTXENT (label and left-out column of a row, see common.h)
  int nblk;              // blocks in use: 2 for the CLIP loss, 1 for the two-view loss and for the symmetric full loss
  const int* gate;       // nullptr: the kernel always runs; else it runs only while *gate == gate_value (the symmetric
  int gate_value;        // full-loss path hands over to the two-block path through this flag)
  int64_t rows, keys;    // the rank's rows and the batch as the caller has them.  The kernels' own b / B arguments are
                         // these rounded up to whole tiles; where they differ (a ragged share), query rows >= rows and
                         // key columns >= keys are padding: X and Y end before it, and who reads tiles of them takes zeros there
};

// Rows of a tile of MOST that exist, of `left` from its first one on (none: a tile that is all padding).
template <int MOST>
__device__ __forceinline__ int rows_there(int64_t left) { return left < 0 ? 0 : left < MOST ? (int)left : MOST; }

__device__ __forceinline__ bool gated_off(const Blocks& bl) { return bl.gate != nullptr && *bl.gate != bl.gate_value; }

__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Positive-pair logit and exponent reference of every local row, one wave per (block, row).  The positive of local row i is
// key row label_row(rank b + i): the same global row for the CLIP loss, the other view's row for the two-view loss.
// B, b: the real sizes; bp: b rounded up to whole tiles (the padding rows get zeros).  The guard takes the positive's norm
// for that of every key, which unit-norm features make true: a pass over all rows for their largest norm costs 10 us of a
// call at B = 32768, d = 512 and 75 at 196608, and k_row_merge finds the rows for which it was not true.  NORMS (symmetric
// path): leaves |x_i| and |y_label| in beta and gdiag, which are free until the merge.
template <bool NORMS>
__global__ __launch_bounds__(256) void k_prep(Blocks bl, int64_t B, int64_t b, int64_t bp, int64_t d, int rank, float s2) {
  if (gated_off(bl)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t rb = (bp + 3) / 4;                      // row workgroups per block
  const BlockPtrs& p = bl.z[blockIdx.x / rb];
  const int64_t i = (blockIdx.x % rb) * 4 + wave;
  if (i >= bp) return;
  if (i >= b) {
    if (lane == 0) { p.zd2[i] = 0.f; p.ref2[i] = 0.f; }
    return;
  }
  const uint16_t* x = p.X + i * d;
  const uint16_t* y = p.Y + label_row((int64_t)rank * b + i, B, bl.variant) * d;
  float dot = 0.f, xx = 0.f, yy = 0.f;
  for (int64_t k = lane * 8; k < d; k += 512) {          // 16-byte pieces (d is a multiple of 8, the rows are 16-byte aligned)
    const u32x4 xw = *reinterpret_cast<const u32x4*>(x + k), yw = *reinterpret_cast<const u32x4*>(y + k);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float x0 = bf16_lo(xw[q]), x1 = bf16_hi(xw[q]), y0 = bf16_lo(yw[q]), y1 = bf16_hi(yw[q]);
      dot = fmaf(x0, y0, dot);
      dot = fmaf(x1, y1, dot);
      xx = fmaf(x0, x0, xx);
      xx = fmaf(x1, x1, xx);
      yy = fmaf(y0, y0, yy);
      yy = fmaf(y1, y1, yy);
    }
  }
  dot = wave_sum(dot);
  xx = sqrtf(wave_sum(xx));
  yy = sqrtf(wave_sum(yy));
  if (lane == 0) {
    p.zd2[i] = s2 * dot;
    p.ref2[i] = fmaxf(s2 * dot, fmaf(fabsf(s2) * xx, yy, -REF_HEADROOM));
    if (NORMS) { p.beta[i] = xx; p.gdiag[i] = yy; }
  }
}

// Element (i, jl) of a stored numerator panel of width W: 16-byte atoms of 8 consecutive keys, by groups of 64 query
// rows, inside a group key piece by key piece (formats FMT_KA / FMT_RA of mfma_tile.h).
// (The definition of the layout; the epilogue below forms the same address piecewise, which the compiler turns into
// a percent faster code than a call of this function.)
__device__ __forceinline__ int64_t e_index(int64_t i, int64_t jl, int64_t W) {
  return ((i >> 6) * (W >> 3) + (jl >> 3)) * 512 + (i & 63) * 8 + (jl & 7);
}

// Epilogue of one logit tile: numerators from the accumulators, row sums, the bf16 numerators to memory.
// Each lane holds, per fragment, 4 consecutive key columns of one query row, lanes l and l + 16 (and l + 32 and l + 48) the two
// halves of 8 consecutive keys; one v_permlane16_swap per register pair of two neighbouring fragments gives every lane a whole
// atom, and 16 lanes (16 consecutive query rows) then store 256 contiguous bytes of the panel (see e_index): no LDS, no barrier, so
// the waves of a workgroup need not meet between the main loops of consecutive tiles.
// MASK_DIAG: the tile contains label columns, which are stored as 0 and kept in fp32 in ediag.
// Local query row i is global row g0 + i; its label is key row label_row(g0 + i), and for the two-view loss its own
// key row g0 + i is left out of its softmax (stored as 0, in no sum), and so are the padding columns from key row
// nkeys (the batch size) on (MASK_EDGE only:
// the caller takes that variant for the tiles they fall into).
// jl0: first key column of the tile relative to the panel of width W that p.E holds.  STREAM: streaming stores
// (past the caches, which keeps the operand tiles in L2; see streaming_stores).  COLS (with STORE): also the lane's sums over its four query
// rows, of each of its keys, of the numerators as stored (col[fragment][r]; padding rows, from row nrows on, are left out under MASK_EDGE).
constexpr int64_t NO_SELF = -((int64_t)1 << 40);

// Do label columns or left-out columns of the T query rows from global row g on fall among key rows [j0, j0 + T)?
// (Only such tiles pay for finding those columns.  The rows of a tile of the two-view loss may lie in both views.)
template <int T>
__device__ __forceinline__ bool tile_has_marked_columns(int64_t g, int64_t B, int variant, int64_t j0) {
  auto hits = [&](int64_t lo, int64_t hi) { return lo < j0 + T && j0 < hi; };       // key rows [lo, hi)
  if (variant != LOSS_NTXENT) return hits(g, g + T);
  const int64_t M = B / 2;
  bool h = hits(g, g + T);                                                           // the rows' own columns
  const int64_t hi1 = g + T < M ? g + T : M;                                         // rows of view one: label g' + M
  if (g < hi1) h = h || hits(g + M, hi1 + M);
  const int64_t lo2 = g > M ? g : M;                                                 // rows of view two: label g' - M
  if (lo2 < g + T) h = h || hits(lo2 - M, g + T - M);
  return h;
}

enum { MASK_NONE = 0, MASK_DIAG = 1, MASK_EDGE = 2 };     // MASK_EDGE: label / left-out columns and padding columns

template <int T, bool STATS, bool STORE, int MASK, bool STREAM = true, bool COLS = false>
__device__ __forceinline__ void logit_epilogue(const BlockPtrs& p, Acc<Cfg<T>::NFA>& acc, int64_t b, float s2, int64_t i0,
                                               int64_t j0, int64_t g0, int variant, int64_t nkeys, const float (&ref2)[4],
                                               int64_t jl0, int64_t W, float (*col)[4] = nullptr, int64_t nrows = 0) {
  constexpr bool DIAG = MASK != MASK_NONE, EDGE = MASK == MASK_EDGE;
  constexpr int WTM = Cfg<T>::WTM, NFA = Cfg<T>::NFA;      // a wave's key columns: 128 (T = 256) or 64
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / Cfg<T>::WN, wn = wave % Cfg<T>::WN, grp = lane >> 4;
  // the wave's first 32 keys of its rows, and in there this lane's atom: row lane % 16, key piece (0, 2, 1, 3)[grp]
  char* e0 = nullptr;
  if (STORE) e0 = const_cast<char*>(uniform_ptr(p.E + (((i0 >> 6) + wn) * (W >> 3) + ((jl0 + wm * WTM) >> 3)) * 512));
  const uint32_t e_lane = (uint32_t)(((grp & 1) << 1 | grp >> 1) * 1024 + (lane & 15) * 16);
  float sums[4];
#pragma unroll
  for (int fn = 0; fn < 4; ++fn) {
    const int il = wn * 64 + fn * 16 + (lane & 15);
    const int64_t i = i0 + il;
    const float ref = ref2[fn];
    // label column of row i, relative to this lane's first key column of the tile (any value outside
    // [0, WTM) means the label is not among this lane's columns)
    const int64_t dl64 = (DIAG ? label_row(g0 + i, nkeys, variant) : 0) - (j0 + wm * WTM + grp * 4);
    const int dl = dl64 >= 0 && dl64 < WTM ? (int)dl64 : -1;
    const int64_t dm64 = (variant == LOSS_NTXENT ? g0 + i : NO_SELF) - (j0 + wm * WTM + grp * 4);
    const int dm = dm64 >= 0 && dm64 < WTM ? (int)dm64 : -1;
    // first padding column, relative like dl (WTM: none among this lane's columns)
    const int64_t jl64 = nkeys - (j0 + wm * WTM + grp * 4);
    const int jlim = jl64 >= WTM ? WTM : jl64 > 0 ? (int)jl64 : 0;
    const bool padding_row = COLS && EDGE && i >= nrows;
    float rowsum = 0.f;
#pragma unroll
    for (int fp = 0; fp < NFA; fp += 2) {
      u32x2 pk[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int fm = fp + q;
        float e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(fmaf(acc[fm][fn][r], s2, -ref));
        if (DIAG) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (dl == fm * 16 + r) {
              if (STATS) p.ediag[i] = e[r];
              e[r] = 0.f;
            }
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (dm == fm * 16 + r || (EDGE && fm * 16 + r >= jlim)) e[r] = 0.f;
        }
        if (STATS) rowsum += (e[0] + e[1]) + (e[2] + e[3]);
        if (STORE) {
          bf16x4 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = (__bf16)e[r];
          pk[q] = __builtin_bit_cast(u32x2, v);
        }
        if (COLS) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float stored = r & 1 ? bf16_hi(pk[q][r >> 1]) : bf16_lo(pk[q][r >> 1]), v = padding_row ? 0.f : stored;
            col[fm][r] = fn == 0 ? v : col[fm][r] + v;
          }
        }
      }
      if (STORE) {
        // lanes 16..31 and 48..63 of the even fragment's registers <-> lanes 0..15 and 32..47 of the odd one's
        const auto w0 = __builtin_amdgcn_permlane16_swap(pk[0][0], pk[1][0], false, false);
        const auto w1 = __builtin_amdgcn_permlane16_swap(pk[0][1], pk[1][1], false, false);
        const u32x4 atom = {w0[0], w1[0], w0[1], w1[1]};
        u32x4* dst = reinterpret_cast<u32x4*>(e0 + fp * 2048 + (e_lane + fn * 256));
        if (STREAM) __builtin_nontemporal_store(atom, dst);
        else *dst = atom;
      }
    }
    if (STATS) {
      rowsum += __shfl_xor(rowsum, 16);
      sums[fn] = rowsum + __shfl_xor(rowsum, 32);
    }
  }
  if (STATS) {
    const float lo = grp & 1 ? sums[1] : sums[0], hi = grp & 1 ? sums[3] : sums[2];
    p.lpart[((T == 256 ? j0 >> 7 : j0 >> 6) + wm) * b + i0 + wn * 64 + lane] = grp & 2 ? hi : lo;
  }
}

// Logit tile + softmax numerators for the key panel [jp0, jp0 + W).  Tile rows (MFMA M side) are key rows
// j, tile columns (N side) are query rows i, so that each lane holds 4 consecutive j of one query row per
// accumulator quad: 8-byte pieces of an E row and an in-lane row sum.
//   STATS: write the partial row sums and the label-column numerator (forward statistics);
//   STORE: write the bf16 numerators to E (panel-relative columns, atom storage, see e_index).
// materialized path: STATS and STORE, one panel = all keys.  fused path: the same for a chunk of rows at a time, or a STATS-only
// pass over all keys (nothing of size b x B is written), then STORE-only passes that recompute one panel at a time.
// b: the rank's rows rounded up to whole tiles; B: the key rows that exist (the panel widths cover them rounded up to
// whole tiles); g0: global row of the rank's first row.  RAGGED: the last key tile may hold padding columns (the
// instance without it keeps the tile walk free of that variant of the epilogue and of the registers it costs).
// Two waves per SIMD, said for both sizes: without it the compiler counts on 512 registers a lane for T = 128, keeps the accumulators
// of the loop that loads in the accumulation file and those of the last K-steps' loop in vector registers, and copies 44 of them there
// and back in every K-step (us: a K-step of a lone workgroup 0.63 / 0.39; a call of B = 1024, N = 4, d = 896 46.2 / 43.1;
// 32768, 8, 64 343 / 336; 2048, 8, 704 46.5 / 44.3).
template <int T, bool STATS, bool STORE, bool RAGGED = false, bool STREAM = true>
__global__ __launch_bounds__(Cfg<T>::NTHREADS, 2) void k_logit_tiles(Blocks bl, int64_t b, int64_t B, int64_t d, int64_t g0, float s2,
                                                          int64_t jp0, int64_t W, int sbi, int sbj, int nblk) {
  if (gated_off(bl)) return;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // Persistent workgroups (one per compute unit) walk the tile lists of the nblk blocks in bl, one after the
  // other, with a stride of the grid size: a wave ends only when all its stores are acknowledged, so ending a
  // workgroup per tile would expose that latency and the launch of the next workgroup once per tile; here a
  // tile's stores drain while the next tile's operands are fetched.  gridDim.x is a multiple of 8, so a
  // workgroup stays on one XCD's contiguous eighth of the tile list.  The list runs over super-blocks of
  // sbi query tiles x sbj key tiles (sbi sbj <= 32; 8 x 4 where the shape allows, see superblock_tile): the
  // workgroups an XCD runs at one time then share sbi + sbj operand tiles in its L2.
  const int nI = (int)(b / T), nJ = (int)(W / T);
  const int total = nI * nJ;
  const int chunk = (total + 7) >> 3, padded = chunk << 3;
  const int lane = threadIdx.x & 63, wn = (threadIdx.x >> 6) % Cfg<T>::WN;
  for (int v = blockIdx.x; v < nblk * padded; v += gridDim.x) {
    const int z = v >= padded ? 1 : 0;
    const int u = v - z * padded;
    const BlockPtrs& p = bl.z[z];
    const int lin = (u & 7) * chunk + (u >> 3);
    if ((u >> 3) >= chunk || lin >= total) continue;                  // padding of the eighths (workgroup-uniform)
    int it, jt;
    superblock_tile(lin, nI, nJ, sbi, sbj, it, jt);
    const int64_t i0 = (int64_t)it * T, j0 = jp0 + (int64_t)jt * T;

    // exponent references of this lane's four query rows, fetched before the main loop so that the loads are
    // not waited for in the epilogue
    float ref2[4];
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) ref2[fn] = p.ref2[i0 + wn * 64 + fn * 16 + (lane & 15)];
    Acc<Cfg<T>::NFA> acc;
#pragma unroll
    for (int i = 0; i < Cfg<T>::NFA; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (RAGGED)
      mainloop<T, FMT_K, FMT_K, true, false, Planes<1, 1>, Bounded>(p.Y + j0 * d, d, p.X + i0 * d, d, (int)(d / BK), smem, acc, T, 0, 0,
                                                                    Bounded{rows_there<T>(B - j0), rows_there<T>(bl.rows - i0), 0u});
    else mainloop<T, FMT_K, FMT_K, true>(p.Y + j0 * d, d, p.X + i0 * d, d, (int)(d / BK), smem, acc);

    // Only the tiles that the label diagonal (or the left-out diagonal) crosses, or that hold padding columns, pay
    // for finding those columns.
    const bool diag = tile_has_marked_columns<T>(g0 + i0, B, bl.variant, j0);
    if (diag || (RAGGED && j0 + T > B)) logit_epilogue<T, STATS, STORE, RAGGED ? MASK_EDGE : MASK_DIAG, STREAM>(p, acc, b, s2, i0, j0, g0, bl.variant, B, ref2, j0 - jp0, W);
    else logit_epilogue<T, STATS, STORE, MASK_NONE, STREAM>(p, acc, b, s2, i0, j0, g0, bl.variant, B, ref2, j0 - jp0, W);
  }
}

constexpr float LN2 = 0.6931471805599453f;

// beta, P_label - 1 and the cross-entropy of row i, from its off-label sum, its label numerator and their total, to memory.
// ce = log(tot / ed); when the label numerator does not dominate it is taken from the exponents,
// log(tot) - z_label ln 2 with z_label = z2_label - ref2, which stays finite when ed itself has underflowed.
__device__ __forceinline__ void row_outputs(const BlockPtrs& p, int64_t i, float off, float ed, float tot, float z_label) {
  p.beta[i] = 1.f / tot;
  p.gdiag[i] = -off / tot;
  p.ce[i] = (ed > 0.5f * tot) ? log1pf(off / ed) : logf(tot) - z_label * LN2;
}

// Xs[k][i] = bf16(scale_i x_ik), kbegin <= k < kend (multiples of 64), for the 64 rows from i0 on, scale = the 64 floats at `scale`
// in LDS (nullptr: 1): the key-side contraction's right operand, with its reduction index contiguous.  All NTH threads
// of the workgroup (256, 512 or 1024), zeros for the rows from `rows` on, 64 x 64 pieces through `tile` (64 x 65 floats of LDS).  The pieces of up to eight
// 64-feature tiles are fetched before the first is turned round, so that their loads are in flight together.
constexpr int TURN_AHEAD = 8;                             // 64-feature tiles fetched together
template <int NTH>
using TurnPieces = u32x2[TURN_AHEAD][1024 / NTH];         // pieces of 4 features per thread and tile

// the pieces of the 64 rows from i0 on (64 rows x 16 pieces a tile), features kc .. of those below kend
template <int NTH>
__device__ __forceinline__ void fetch_rows(const BlockPtrs& p, int64_t rows, int64_t d, int64_t kc, int64_t kend, int64_t i0, TurnPieces<NTH>& w) {
#pragma unroll
  for (int a = 0; a < TURN_AHEAD; ++a)
    if (kc + a * 64 < kend)
#pragma unroll
      for (int q = 0; q < 1024 / NTH; ++q) {
        const int e = threadIdx.x + q * NTH, r = e >> 4, c4 = (e & 15) * 4;
        w[a][q] = u32x2{0u, 0u};
        if (i0 + r < rows) w[a][q] = *reinterpret_cast<const u32x2*>(p.X + (i0 + r) * d + kc + a * 64 + c4);
      }
}
template <int NTH>
__device__ __forceinline__ void turn_rows(const BlockPtrs& p, int64_t b, int64_t kc, int64_t kend, int64_t i0, const float* scale, float (*tile)[65], const TurnPieces<NTH>& w) {
  const int t = threadIdx.x;
#pragma unroll
  for (int a = 0; a < TURN_AHEAD; ++a) {
    const int64_t k0 = kc + a * 64;
    if (k0 >= kend) break;
    __syncthreads();                                      // the tile's previous contents have been read
#pragma unroll
    for (int q = 0; q < 1024 / NTH; ++q) {
      const int e = t + q * NTH, r = e >> 4, c4 = (e & 15) * 4;
      const float sc = scale ? scale[r] : 1.f;
      tile[r][c4 + 0] = sc * bf16_lo(w[a][q][0]);
      tile[r][c4 + 1] = sc * bf16_hi(w[a][q][0]);
      tile[r][c4 + 2] = sc * bf16_lo(w[a][q][1]);
      tile[r][c4 + 3] = sc * bf16_hi(w[a][q][1]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 1024 / NTH; ++q) {                // 64 features x 16 pieces of 4 rows
      const int e = t + q * NTH, k = e >> 4, i4 = (e & 15) * 4;
      bf16x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (__bf16)tile[i4 + j][k];
      *reinterpret_cast<bf16x4*>(p.Xs + (k0 + k) * b + i0 + i4) = v;
    }
  }
}
template <int NTH>
__device__ __forceinline__ void scale_transpose_rows(const BlockPtrs& p, int64_t rows, int64_t b, int64_t d, int64_t kbegin, int64_t kend, int64_t i0, const float* scale,
                                                     float (*tile)[65]) {
  for (int64_t kc = kbegin; kc < kend; kc += 64 * TURN_AHEAD) {
    TurnPieces<NTH> w;
    fetch_rows<NTH>(p, rows, d, kc, kend, i0, w);
    turn_rows<NTH>(p, b, kc, kend, i0, scale, tile, w);
  }
}

// The statistics of 64 rows redone by the workgroup of k_row_merge that found one whose total is lost (inputs that are not
// CLIP-like): a first sweep over all keys finds every row's true maximum logit, its new exponent reference, a second forms the
// numerators (stored to E if `store`) and the row sums against it.  Wave w takes the key strips w, w + 16, ... of 32 keys
// against all 64 rows, in 16 x 16 x 32 blocks, key rows on the M side as in the logit kernel.  What bounds it is the lines of
// the features it asks for: so the rows' go through LDS, 64 features at a time (`xt`: two such pieces, 16 KiB, 16-byte chunks
// XOR-swizzled with the row), and a key's come straight from memory, a whole line at once.  (All rows redone, features of norm 4
// to 8 at B = 32768, d = 512: a call takes 2.9 ms at N = 8 and 2.35 at N = 64; with both operands' fragments straight from
// memory and every workgroup on the same rows at it, 6.1 and 5.5; a call that redoes none 0.75 and 0.145.)
// Local rows i0 .. i0 + 63, of which those from `rows` on are padding, global row g0 + i; Bp: the keys rounded up to whole tiles.  Leaves the rows' sums in
// off_s and their label numerators in ed_s.
__device__ __forceinline__ void redo_rows(const BlockPtrs& p, int variant, int64_t rows, int64_t keys, int64_t Bp, int64_t d, int64_t i0, int64_t g0, float s2, bool store,
                                       float (*red)[64], float* ref_s, float* off_s, float* ed_s, char* xt) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, l16 = lane & 15, grp = lane >> 4;
  const uint32_t row_bytes = (uint32_t)d * 2;
  const char* xb = uniform_ptr(p.X + i0 * d);                                      // threads 0 .. 511: row t / 8, chunk t % 8 of a piece
  const uint32_t x_off = (uint32_t)(t >> 3) * row_bytes + (t & 7) * 16;
  const uint32_t x_put = (uint32_t)((t >> 3) * 128 + (((t & 7) ^ ((t >> 3) & 7)) << 4));
  const bool x_there = t < 512 && i0 + (t >> 3) < rows;
  int buf = 0;
  f32x4 acc[2][4];                                        // [16 keys][16 rows]; a lane: keys 4 grp .. + 3 of row l16
  auto strip = [&](int j0) {                              // (all waves together)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char* yb = uniform_ptr(p.Y + (int64_t)j0 * d);
    uint32_t y_off[2];                                    // of a lane's piece from the strip's first key; the last key for those past it
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = 16 * u + l16, most = (int)keys - 1 - j0;
      y_off[u] = (uint32_t)(r < most ? r : most) * row_bytes + grp * 16;
    }
    u32x4 next = {0u, 0u, 0u, 0u};
    if (x_there) next = *reinterpret_cast<const u32x4*>(xb + x_off);
#pragma unroll 1
    for (uint32_t k = 0; k < row_bytes; k += 128) {
      bf16x8 a[2][2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h) a[h][u] = *reinterpret_cast<const bf16x8*>(yb + (k + 64 * h) + y_off[u]);
      char* piece = xt + buf * 8192;
      buf ^= 1;
      if (t < 512) {
        *reinterpret_cast<u32x4*>(piece + x_put) = next;
        if (x_there && k + 128 < row_bytes) next = *reinterpret_cast<const u32x4*>(xb + x_off + k + 128);
      }
      lds_barrier();                                      // (the other piece: read before the previous barrier, written after it)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bf16x8 q = *reinterpret_cast<const bf16x8*>(piece + (v * 16 + l16) * 128 + (((h * 4 + grp) ^ (l16 & 7)) << 4));
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[h][u], q, acc[u][v], 0, 0, 0);
        }
    }
  };
  float m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll 1
  for (int base = 0; base < (int)keys; base += 16 * 32) {
    const int j0 = base + wave * 32;
    strip(j0 < (int)keys ? j0 : 0);                       // a wave without a strip works on the first one and drops it
    if (j0 >= (int)keys) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int self = (int)masked_col(g0 + i0 + v * 16 + l16, variant);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = j0 + u * 16 + grp * 4 + e;
          if (j < (int)keys && j != self) m[v] = fmaxf(m[v], acc[u][v][e] * s2);
        }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    m[v] = fmaxf(m[v], __shfl_xor(m[v], 16));
    m[v] = fmaxf(m[v], __shfl_xor(m[v], 32));
    if (grp == 0) red[wave][v * 16 + l16] = m[v];
  }
  __syncthreads();
  if (wave == 0) {
    float r = red[0][lane];
    for (int w = 1; w < 16; ++w) r = fmaxf(r, red[w][lane]);
    ref_s[lane] = r;
    p.ref2[i0 + lane] = r;
  }
  __syncthreads();
  float rs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int base = 0; base < (int)keys; base += 16 * 32) {
    const int j0 = base + wave * 32;
    strip(j0 < (int)keys ? j0 : 0);
    if (j0 >= (int)keys) continue;
    // (element (row, key) of the group is at e_index: scalar base of the strip plus this lane's place in it)
    char* erow = const_cast<char*>(uniform_ptr(p.E + e_index(i0, j0, Bp))) + (uint32_t)(((grp >> 1) * 512 + l16 * 8 + (grp & 1) * 4) * 2);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = v * 16 + l16;
      const int64_t g = g0 + i0 + row;
      const int label = (int)label_row(g, keys, variant), self = (int)masked_col(g, variant);
      const float ref = ref_s[row];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = j0 + u * 16 + grp * 4;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float n = j + e < (int)keys && j + e != self ? __builtin_amdgcn_exp2f(fmaf(acc[u][v][e], s2, -ref)) : 0.f;
          if (j + e == label) { ed_s[row] = n; n = 0.f; }
          rs[v] += n;
          o[e] = (__bf16)n;
        }
        if (store) *reinterpret_cast<bf16x4*>(erow + (u * 1024 + v * 128) * 2) = o;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    rs[v] += __shfl_xor(rs[v], 16);
    rs[v] += __shfl_xor(rs[v], 32);
    if (grp == 0) red[wave][v * 16 + l16] = rs[v];
  }
  __syncthreads();
  if (wave == 0) {
    float r = red[0][lane];
    for (int w = 1; w < 16; ++w) r += red[w][lane];
    off_s[lane] = r;
  }
  __syncthreads();
}

// What k_row_merge needs besides the blocks.
struct MergeShape {
  int64_t b, Bp, d;                // rows and key rows in memory (whole tiles)
  int64_t g0;                      // global row of the rank's first row
  int nparts0, nparts1;            // partial sums per row of block 0 / block 1
  int store;                       // redone rows: numerators to E
  int fchunks;                     // go on to write the rows of Xs = (beta x)^T, by this many workgroups (grid.z); 0: not
  float s2;
  const float* global_ref;         // symmetric full loss: the one exponent reference every row shares
  int* bad_flag;                   // and where that path records that a row or column total was lost (nullptr: rows are redone)
};

// Row totals -> beta, P_label - 1, cross-entropy.  A workgroup takes 64 rows; its 16 waves each add a
// sixteenth of the column parts (lane = row, so the reads are coalesced), combined in fixed order.  A small share has few
// such workgroups, each of which would turn round all of its rows' features: fchunks of them then share the features of
// the same rows, and all but the first add up the totals for themselves only (b = 512, d = 512: 9.3 -> 6.8 us with eight).
// Latencies bound it: the features and the row's own values do not wait for the totals (us a call: B = 4096, N = 16, d = 192 35.1 -> 33.0; 5072,
// 16, 256 40.2 -> 38.7; 2048, 2, 320 43.2 -> 42.4; of 39 random calls of 33 to 540 us 1 % in the mean).
__global__ __launch_bounds__(1024) void k_row_merge(Blocks bl, MergeShape f) {
  if (gated_off(bl)) return;
  const int64_t b = f.b;
  const int nparts = blockIdx.y ? f.nparts1 : f.nparts0;
  __shared__ float red[16][64];
  __shared__ float beta_s[64], ref_s[64], off_s[64], ed_s[64];
  __shared__ int redo, over[16];
  __shared__ __attribute__((aligned(16))) float tile[64][65];
  const BlockPtrs& p = bl.z[blockIdx.y];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * 64, i = i0 + lane;
  // The features that the end of the kernel turns round and what wave 0 needs of a row, asked for before the totals.
  const int64_t per = f.fchunks ? (f.d / 64 + f.fchunks - 1) / f.fchunks * 64 : 0, kz = blockIdx.z * per, kend = kz + per < f.d ? kz + per : f.d;
  TurnPieces<1024> w;
  if (f.fchunks) fetch_rows<1024>(p, bl.rows, f.d, kz, kend, i0, w);
  float ed0 = 0.f, zd = 0.f, ref = 0.f;
  if (wave == 0) {
    ed0 = p.ediag[i];
    zd = p.zd2[i];
    ref = f.global_ref ? *f.global_ref : p.ref2[i];
  }
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f, most = 0.f;           // most: the row's largest part
  int q = wave;
  for (; q + 112 < nparts; q += 128) {                   // eight loads in flight
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p.lpart[(int64_t)(q + 16 * u) * b + i];
    a0 += v[0]; a1 += v[1]; a2 += v[2]; a3 += v[3];
    a0 += v[4]; a1 += v[5]; a2 += v[6]; a3 += v[7];
#pragma unroll
    for (int u = 0; u < 8; ++u) most = fmaxf(most, v[u]);
  }
  for (; q + 48 < nparts; q += 64) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p.lpart[(int64_t)(q + 16 * u) * b + i];
    a0 += v[0]; a1 += v[1]; a2 += v[2]; a3 += v[3];
#pragma unroll
    for (int u = 0; u < 4; ++u) most = fmaxf(most, v[u]);
  }
  for (; q < nparts; q += 16) {
    const float v = p.lpart[(int64_t)q * b + i];
    a0 += v;
    most = fmaxf(most, v);
  }
  red[wave][lane] = (a0 + a1) + (a2 + a3);
  const int wave_over = __any(most > ROW_PART_MAX);
  if (lane == 0) over[wave] = wave_over;
  __syncthreads();
  // wave 0, lane = row: outputs of the row from its off-label sum and its label numerator; is the total lost?  (One that is not
  // a number comes from features that are not, or from logits past fp32: no other reference of the row's helps.)
  const bool writer = blockIdx.z == 0;                  // of several workgroups on the same rows
  auto finish = [&](float off, float ed) {
    if (i >= bl.rows) {                                 // a padding row: no weight anywhere
      if (writer) { p.ref2[i] = 0.f; p.beta[i] = 0.f; p.gdiag[i] = 0.f; p.ce[i] = 0.f; }
      beta_s[lane] = 0.f;
      return false;
    }
    const float tot = off + ed;
    beta_s[lane] = 1.f / tot;
    if (writer) row_outputs(p, i, off, ed, tot, zd - ref);
    return f.bad_flag ? !(tot >= ROW_TOTAL_FLOOR) : tot < ROW_TOTAL_FLOOR;
  };
  if (wave == 0) {
    float off = 0.f;
#pragma unroll
    for (int w = 0; w < 16; w += 4) off += (red[w][lane] + red[w + 1][lane]) + (red[w + 2][lane] + red[w + 3][lane]);
    if (f.global_ref && writer) p.ref2[i] = ref;
    const bool lost = __any(finish(off, ed0)), above = __any(lane < 16 && over[lane & 15]);
    if (lane == 0) {
      redo = (lost || above) && !f.bad_flag;
      if (lost && f.bad_flag) *f.bad_flag = 1;
    }
  }
  __syncthreads();
  if (redo) {                                           // by the first of the workgroups on these rows, which goes on to all of their features
    if (!writer) return;
    redo_rows(p, bl.variant, bl.rows, bl.keys, f.Bp, f.d, i0, f.g0, f.s2, f.store, red, ref_s, off_s, ed_s, reinterpret_cast<char*>(tile));
    if (wave == 0) {
      ref = ref_s[lane];
      finish(off_s[lane], ed_s[lane]);
    }
    __syncthreads();
    if (f.fchunks) scale_transpose_rows<1024>(p, bl.rows, b, f.d, 0, f.d, i0, beta_s, tile);
    return;
  }
  if (f.fchunks) {
    turn_rows<1024>(p, b, kz, kend, i0, beta_s, tile, w);
    scale_transpose_rows<1024>(p, bl.rows, b, f.d, kz + 64 * TURN_AHEAD, kend, i0, beta_s, tile);
  }
}

// Xs = X^T for one block without any scaling (the symmetric full loss folds both normalisations into the stored
// matrix instead): a workgroup per 64 rows.
__global__ __launch_bounds__(1024) void k_transpose(Blocks bl, int64_t b, int64_t d) {
  if (gated_off(bl)) return;
  __shared__ float tile[64][65];
  scale_transpose_rows<1024>(bl.z[0], bl.rows, b, d, 0, d, (int64_t)blockIdx.x * 64, nullptr, tile);
}

// The two gradient contractions of every block, in one launch: they are independent of each other, so where neither has
// the workgroups to fill the chip they fill it together, and neither waits for the other's last workgroups (one launch
// against two: 56 us against 68 a call at b = 512, B = 1024, d = 256; 4060 against 4098 for the symmetric B = 32768).
// blockIdx.x < q_wgs: query-side workgroups, the rest key-side ones (q_wgs is a multiple of 8, so that both parts keep
// their workgroup -> XCD mapping).
//
// Key side, without its label-column term: gk[j][k] (+)= cs * sum_i E[i][j] Xs[k][i].
// (The term [j = label_i] gdiag_i x_ik is added by the finalize kernel, which owns the rank's rows.)
// GEMM M = key rows j (operand E read transposed), N = feature index k, reduction over the rank's rows.
// KMODE: KEY_WRITE / KEY_ADD overwrite gk / add to it; KEY_SPLIT leaves the unscaled sums of key_splits ranges of the rows
// in kpart for the finalize kernel (wanted where B x d has too few tiles and the rank many rows).
//
// Query side, split over the key index: part[ks][i][k] = sum_{j in split ks} E[i][j] y_jk.
// GEMM M = query rows i, N = feature index k (operand Y read transposed), reduction over key rows.
// A "slice" is one (z, ks): all its workgroups read the same rows of Y, so slices are pinned to XCDs (workgroups are dealt
// round-robin to the 8 XCDs): with S = nblk splitk slices, either S/8 slices per XCD one after the other (S a multiple of
// 8), or 8/S XCDs per slice sharing its tiles (S divides 8).  Then Y comes in from the fabric once per slice instead
// of once per XCD.  Any other S falls back to slices laid out contiguously.
struct GradShape {
  int64_t b, B, d, jp0, W;          // b, B: rounded up to whole tiles; key panel [jp0, jp0 + W)
  int nMq, nMk, nN;                 // row tiles of the query and key sides, column tiles
  int splitk, ktps;                 // query side: splits of the W keys, K-steps per split
  int key_splits, key_ktps;         // key side: splits of the b rows, K-steps per split
  int q_wgs;
};
enum { KEY_WRITE = 0, KEY_ADD = 1, KEY_SPLIT = 2 };

// RAGGED: the last of the W key rows may not exist; the query side reads zeros there, which meet the zeros of the numerators' padding columns.
template <int T, int KMODE, bool QADD, bool RAGGED>
__global__ __launch_bounds__(Cfg<T>::NTHREADS) void k_grads(Blocks bl, GradShape g, float cs) {
  if (gated_off(bl)) return;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int64_t b = g.b, d = g.d, W = g.W;
  Acc<Cfg<T>::NFA> acc;
  if ((int)blockIdx.x < g.q_wgs) {
    const int tiles = g.nMq * g.nN, S = bl.nblk * g.splitk;
    const int w = blockIdx.x, xcd = w & 7, r = w >> 3;
    int slice, tile;
    if (S % 8 == 0) {
      slice = xcd + 8 * (r / tiles);
      tile = r % tiles;
    } else if (8 % S == 0) {
      const int G = 8 / S;
      slice = xcd % S;
      tile = xcd / S + G * r;
    } else {
      slice = w / tiles;
      tile = w % tiles;
    }
    if (slice >= S || tile >= tiles) return;
    const BlockPtrs& p = bl.z[slice / g.splitk];
    const int ks = slice % g.splitk;
    const int nt = tile % g.nN, mt = tile / g.nN;
    const int64_t i0 = (int64_t)mt * T, k0 = (int64_t)nt * T;
    const int kt_total = (int)(W / BK);
    const int kt0 = ks * g.ktps;
    int kts = kt_total - kt0;
    if (kts > g.ktps) kts = g.ktps;
    const int ncols = d - k0 < T ? (int)(d - k0) : T;               // the last column tile may be partial (d % 64 == 0)
    // (kts >= 1: the plan's split count is the number of splits that hold at least one K-step)
    const uint16_t* Eq = p.E + ((i0 >> 6) * (W >> 6) + kt0) * 4096;
    const int64_t j0 = g.jp0 + (int64_t)kt0 * BK;
    if constexpr (RAGGED)
      mainloop<T, FMT_KA, FMT_R, false, true, Planes<1, 1>, Bounded>(Eq, (W >> 6) * 4096, p.Y + j0 * d + k0, d, kts, smem, acc, ncols, 0, 0,
                                                                     Bounded{0, rows_there<(1 << 30)>(bl.keys - j0), (uint32_t)(k0 * 2)});
    else mainloop<T, FMT_KA, FMT_R, false, true>(Eq, (W >> 6) * 4096, p.Y + j0 * d + k0, d, kts, smem, acc, ncols);
    store_tile_f32<T, QADD>(acc, smem, p.part + (int64_t)ks * b * d + i0 * d + k0, d, 1.0f, ncols);
    return;
  }
  const int tiles = g.nMk * g.nN * g.key_splits, per_block = (tiles + 7) / 8 * 8;
  const int w = blockIdx.x - g.q_wgs, z = w / per_block;
  int lin;
  if (!xcd_linear(w - z * per_block, tiles, lin)) return;
  const BlockPtrs& p = bl.z[z];
  const int nt = lin % g.nN, t2 = lin / g.nN, mt = t2 % g.nMk, ks = t2 / g.nMk;
  const int64_t jl0 = (int64_t)mt * T, k0 = (int64_t)nt * T;        // key rows jp0 + jl0 .. of the panel
  const int ncols = d - k0 < T ? (int)(d - k0) : T;
  const int kt0 = ks * g.key_ktps;
  int kts = (int)(b / BK) - kt0;
  if (kts > g.key_ktps) kts = g.key_ktps;
  mainloop<T, FMT_RA, FMT_K, false, true>(p.E + (jl0 >> 6) * 4096 + (int64_t)kt0 * (W >> 6) * 4096, (W >> 6) * 4096,
                                          p.Xs + k0 * b + (int64_t)kt0 * BK, b, kts, smem, acc, ncols);
  const int64_t left = bl.keys - (g.jp0 + jl0);                      // key rows that exist from this tile's first one on
  float* out = KMODE == KEY_SPLIT ? p.kpart + ((int64_t)ks * g.B + jl0) * d + k0 : p.gk + (g.jp0 + jl0) * d + k0;
  store_tile_f32<T, KMODE == KEY_ADD>(acc, smem, out, d, KMODE == KEY_SPLIT ? 1.0f : cs, ncols, left < T ? (int)left : T);
}

// u[n]: sum over the split-K slices ks0, ks0 + step, ... (< splitk), in that order, of the 16-byte piece at from[n], slices `pitch` elements
// apart.  DEPTH slices of every piece are in flight at a time, the last ones too (a plain loop waits for every load).
template <int N, int DEPTH = 4>
__device__ __forceinline__ void sum_slices(const float* const (&from)[N], int64_t pitch, int ks0, int step, int splitk, f32x4 (&u)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) u[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int ks = ks0; ks < splitk; ks += DEPTH * step) {
    f32x4 v[DEPTH][N];
#pragma unroll
    for (int q = 0; q < DEPTH; ++q) {
      const int at = ks + q * step;
#pragma unroll
      for (int n = 0; n < N; ++n) {
        v[q][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (at < splitk) v[q][n] = *reinterpret_cast<const f32x4*>(from[n] + at * pitch);
      }
    }
#pragma unroll
    for (int q = 0; q < DEPTH; ++q)
#pragma unroll
      for (int n = 0; n < N; ++n) u[n] += v[q][n];
  }
}

// What the finalize kernels add up for a row, besides its own terms.
struct FinalizeShape {
  int64_t b, bp;        // the rank's rows (of the chunk); row pitch of part
  int64_t B, Bp;        // all rows; row pitch of kpart
  int64_t d;
  int64_t g0;           // global row of the first of them
  int splitk, key_splits, accumulate;
};

// Everything that lands in the rank's own rows, for both blocks at once.  With lab = label of local row i:
//   gI[lab] += cs (beta^A_i sum_ks part^A + gdiag^A_i T[lab])    query side of block A (Eq. 4)
//            + cs gdiag^C_i T[lab]                                label-column term of block C's key side
//   gT[lab] += cs (beta^C_i sum_ks part^C + gdiag^C_i I[lab]) + cs gdiag^A_i I[lab]
// and the rows' shares of d/ds, <query-side vector, x_i>, per block.  Fixed summation order.
// KSPLIT (the key-side contraction was split, k_grads<.., KEY_SPLIT>): the kernel runs over all B rows and starts each from
//   gI[j] = [accumulate] gI[j] + cs sum_ks kpart^C[ks][j],  gT[j] likewise from kpart^A.
// One wave per row: memory's rate bounds it, so what counts is how many waves fit (64 registers; with the loads below 108, and 22.2 us
// instead of 20.6 at b = 4096, B = 32768, d = 512).  ROWWG (few rows, where rows / 4 workgroups would leave most of the chip idle while
// each wave walks all the split-K slices): one workgroup per row, its four waves each add every fourth slice and wave 0 combines them.
// Latencies one after the other bound that: both blocks' slices, P pieces of columns (2 for d > 256, where the key side is not split as well) and
// what they are added to are asked for together (b = 512, d = 1024 13.8 -> 11.3 us; 257, 768 8.7 -> 6.8; calls of B = 15040, N = 64,
// d = 640 79.6 -> 76.4, 12864, 64, 768 154.9 -> 148.9, 3536, 8, 384 44.0 -> 42.6; of 70 random calls of 40 to 400 us 1 % in the mean).
template <bool ROWWG, bool KSPLIT, int P>
__global__ __launch_bounds__(256, P == 2 ? 3 : ROWWG ? 4 : 1) void k_finalize(Blocks bl, FinalizeShape f, float cs) {
  if (gated_off(bl)) return;
  constexpr int NSUM = KSPLIT ? 4 : 2;                   // sums per piece of 256 columns
  __shared__ f32x4 others[ROWWG ? 3 : 1][P][NSUM][64];
  const BlockPtrs& pa = bl.z[0];
  const BlockPtrs& pc = bl.z[1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = ROWWG ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
  if (row >= (KSPLIT ? f.B : f.b)) return;              // ROWWG: the whole workgroup
  const int64_t i = KSPLIT ? row - f.g0 : row;         // local row
  const int64_t lab = KSPLIT ? row : f.g0 + row;       // global row
  const bool own = !KSPLIT || (i >= 0 && i < f.b);
  float beta_a = 0.f, gd_a = 0.f, beta_c = 0.f, gd_c = 0.f;
  if (own) { beta_a = pa.beta[i]; gd_a = pa.gdiag[i]; beta_c = pc.beta[i]; gd_c = pc.gdiag[i]; }
  const int64_t d = f.d;
  const int first = ROWWG ? wave : 0, step = ROWWG ? 4 : 1;
  float dot_a = 0.f, dot_c = 0.f;
  for (int64_t kc = 0; kc < d; kc += 256 * P) {
    f32x4 gi[P], gt[P];                                  // what the sums are added to
    u32x2 iw[P], tw[P];                                  // I[lab], T[lab]
    auto fetch = [&](int h) {
      const int64_t k = kc + h * 256 + lane * 4;
      gi[h] = f32x4{0.f, 0.f, 0.f, 0.f}; gt[h] = f32x4{0.f, 0.f, 0.f, 0.f};
      iw[h] = u32x2{0u, 0u}; tw[h] = u32x2{0u, 0u};
      if (k < d && (!ROWWG || wave == 0)) {
        if (!KSPLIT || f.accumulate) {
          gi[h] = *reinterpret_cast<f32x4*>(pa.gq + lab * d + k);
          gt[h] = *reinterpret_cast<f32x4*>(pc.gq + lab * d + k);
        }
        if (own) {
          iw[h] = *reinterpret_cast<const u32x2*>(pa.X + i * d + k);
          tw[h] = *reinterpret_cast<const u32x2*>(pc.X + i * d + k);
        }
      }
    };
    if (ROWWG)                                           // few rows: their loads before the sums'
#pragma unroll
      for (int h = 0; h < P; ++h) fetch(h);
    f32x4 u[P][NSUM];                                    // query side of A and C, key side of A and C
    auto sums = [&](auto pieces) {
      constexpr int H = decltype(pieces)::value;
      auto two = [&](const float* a, const float* c, int64_t r, int64_t pitch, int splits, int at) {
        const float* from[2 * H];
        f32x4 s[2 * H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int64_t k = kc + h * 256 + lane * 4, there = r * d + (k < d ? k : 0);
          from[2 * h] = a + there;
          from[2 * h + 1] = c + there;
        }
        if constexpr (ROWWG) {
          sum_slices<2 * H, H == 1 ? 4 : 2>(from, pitch * d, first, step, splits, s);
        } else {                                         // (one after the other: the kernel is at memory's rate, by the waves that fit)
#pragma unroll
          for (int n = 0; n < 2 * H; ++n) {
            f32x4 one[1];
            sum_slices<1>({from[n]}, pitch * d, first, step, splits, one);
            s[n] = one[0];
          }
        }
#pragma unroll
        for (int h = 0; h < H; ++h) { u[h][at] = s[2 * h]; u[h][at + 1] = s[2 * h + 1]; }
      };
      if (own) {
        two(pa.part, pc.part, i, f.bp, f.splitk, 0);
      } else {
#pragma unroll
        for (int h = 0; h < H; ++h) u[h][0] = u[h][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if constexpr (KSPLIT) two(pa.kpart, pc.kpart, row, f.Bp, f.key_splits, 2);
    };
    const bool more = P > 1 && kc + 256 < d;             // (workgroup-uniform) a second piece of columns
    if (more) sums(std::integral_constant<int, P>{});
    else sums(std::integral_constant<int, 1>{});
#pragma unroll
    for (int h = 0; h < P; ++h) {
      if (h > 0 && !more) break;
      if (ROWWG) {
        if (wave > 0)
#pragma unroll
          for (int q = 0; q < NSUM; ++q) others[wave - 1][h][q][lane] = u[h][q];
      }
    }
    if (ROWWG) __syncthreads();
#pragma unroll
    for (int h = 0; h < P; ++h) {
      const int64_t k = kc + h * 256 + lane * 4;
      if ((ROWWG && wave > 0) || k >= d) continue;
      if (!ROWWG) fetch(h);
      if (ROWWG)
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
          for (int q = 0; q < NSUM; ++q) u[h][q] += others[w][h][q][lane];
      if constexpr (KSPLIT) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { gt[h][e] = fmaf(cs, u[h][2][e], gt[h][e]); gi[h][e] = fmaf(cs, u[h][3][e], gi[h][e]); }
      }
      if (own) {
        const float iv[4] = {bf16_lo(iw[h][0]), bf16_hi(iw[h][0]), bf16_lo(iw[h][1]), bf16_hi(iw[h][1])};
        const float tv[4] = {bf16_lo(tw[h][0]), bf16_hi(tw[h][0]), bf16_lo(tw[h][1]), bf16_hi(tw[h][1])};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ga = fmaf(beta_a, u[h][0][e], gd_a * tv[e]);
          const float gc = fmaf(beta_c, u[h][1][e], gd_c * iv[e]);
          gi[h][e] = fmaf(cs * gd_c, tv[e], fmaf(cs, ga, gi[h][e]));
          gt[h][e] = fmaf(cs * gd_a, iv[e], fmaf(cs, gc, gt[h][e]));
          dot_a = fmaf(ga, iv[e], dot_a);
          dot_c = fmaf(gc, tv[e], dot_c);
        }
      }
      *reinterpret_cast<f32x4*>(pa.gq + lab * d + k) = gi[h];
      *reinterpret_cast<f32x4*>(pc.gq + lab * d + k) = gt[h];
    }
    if (ROWWG && kc + 256 * P < d) __syncthreads();      // read before the next pieces overwrite it
  }
  if (!own || (ROWWG && wave > 0)) return;
  dot_a = wave_sum(dot_a);
  dot_c = wave_sum(dot_c);
  if (lane == 0) { pa.rowds[i] = dot_a; pc.rowds[i] = dot_c; }
}

// up to this many rows finalize with one workgroup per row
constexpr int64_t FINALIZE_ROWWG_MAX = 1024;

// The same for the two-view loss (one block, X = Y = Z, gq = gk = gZ).  With g = rank b + i the row's own global row
// and lab its positive's row:
//   gZ[g]   += cs (beta_i sum_ks part + gdiag_i Z[lab])     query side
//   gZ[lab] += cs gdiag_i Z[g]                              label-column term of the key side
// The second line lands in another row, lab.  If lab belongs to this rank too, the wave that owns it adds the term
// (seen from there it reads gdiag_i' Z[lab'] with i' its positive, since the positive of the positive is the row
// itself); otherwise the wave of row i writes it.  Every row of gZ so has exactly one writer in this kernel.
// KSPLIT: the kernel runs over all B rows as above, every row adds what its positive owes it and nobody writes
// another's row.
template <bool KSPLIT>
__global__ __launch_bounds__(256) void k_finalize_ntxent(Blocks bl, FinalizeShape f, float cs) {
  if (gated_off(bl)) return;
  const BlockPtrs& p = bl.z[0];
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= (KSPLIT ? f.B : f.b)) return;
  const int64_t i = KSPLIT ? row - f.g0 : row;
  const int64_t g = KSPLIT ? row : f.g0 + row, lab = label_row(g, f.B, LOSS_NTXENT);
  const bool own = !KSPLIT || (i >= 0 && i < f.b);
  const int64_t ip = lab - f.g0;                     // local index of the positive, if it is local
  const bool pos_local = ip >= 0 && ip < f.b;
  const bool owes = !KSPLIT && !pos_local;                            // this wave writes its term into row lab
  const float beta = own ? p.beta[i] : 0.f, gd = own ? p.gdiag[i] : 0.f, gd_pos = pos_local ? p.gdiag[ip] : 0.f;
  const uint16_t* Zfull = p.Y;
  const int64_t d = f.d;
  float dot = 0.f;
  for (int64_t k = lane * 4; k < d; k += 256) {
    f32x4 u[1] = {{0.f, 0.f, 0.f, 0.f}}, kv[1];
    auto query_side = [&] { sum_slices<1>({p.part + i * d + k}, f.bp * d, 0, 1, f.splitk, u); };
    if (!KSPLIT) query_side();
    const u32x2 zw = *reinterpret_cast<const u32x2*>(Zfull + g * d + k);        // Z[g]
    const u32x2 pw = *reinterpret_cast<const u32x2*>(Zfull + lab * d + k);      // Z[lab]
    const float zv[4] = {bf16_lo(zw[0]), bf16_hi(zw[0]), bf16_lo(zw[1]), bf16_hi(zw[1])};
    const float pv[4] = {bf16_lo(pw[0]), bf16_hi(pw[0]), bf16_lo(pw[1]), bf16_hi(pw[1])};
    f32x4 mine = {0.f, 0.f, 0.f, 0.f}, oth = {0.f, 0.f, 0.f, 0.f};
    if (!KSPLIT || f.accumulate) mine = *reinterpret_cast<f32x4*>(p.gq + g * d + k);
    if (owes) oth = *reinterpret_cast<f32x4*>(p.gq + lab * d + k);
    if constexpr (KSPLIT) {
      if (own) query_side();
      sum_slices<1>({p.kpart + row * d + k}, f.Bp * d, 0, 1, f.key_splits, kv);
#pragma unroll
      for (int e = 0; e < 4; ++e) mine[e] = fmaf(cs, kv[0][e], mine[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ga = fmaf(beta, u[0][e], gd * pv[e]);
      mine[e] = fmaf(cs * gd_pos, pv[e], fmaf(cs, ga, mine[e]));      // + what the local positive owes this row
      oth[e] = fmaf(cs * gd, zv[e], oth[e]);
      dot = fmaf(ga, zv[e], dot);
    }
    *reinterpret_cast<f32x4*>(p.gq + g * d + k) = mine;
    if (owes) *reinterpret_cast<f32x4*>(p.gq + lab * d + k) = oth;
  }
  if (!own) return;
  dot = wave_sum(dot);
  if (lane == 0) p.rowds[i] = dot;
}

// loss_r = c sum ce, gs_r = c sum rowds over the blocks of the loss; one workgroup, fixed order.
__global__ __launch_bounds__(1024) void k_scalars(Blocks bl, int64_t b, float c, int accumulate, float* loss, float* gs) {
  if (gated_off(bl)) return;
  __shared__ float ra[16], rg[16];
  float a = 0.f, g = 0.f;
  for (int z = 0; z < bl.nblk; ++z)
    for (int64_t i0 = threadIdx.x; i0 < b; i0 += 4096) {              // four loads of each array in flight
      float c[4], r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u * 1024;
        c[u] = i < b ? bl.z[z].ce[i] : 0.f;
        r[u] = i < b ? bl.z[z].rowds[i] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { a += c[u]; g += r[u]; }
    }
  a = wave_sum(a);
  g = wave_sum(g);
  if ((threadIdx.x & 63) == 0) { ra[threadIdx.x >> 6] = a; rg[threadIdx.x >> 6] = g; }
  __syncthreads();
  if (threadIdx.x == 0) {
    float sa = 0.f, sg = 0.f;
    for (int w = 0; w < 16; ++w) { sa += ra[w]; sg += rg[w]; }
    *loss = (accumulate ? *loss : 0.f) + c * sa;
    *gs = (accumulate ? *gs : 0.f) + c * sg;
  }
}

// ------------------------------------------------------------------------------------------------
// Symmetric full loss (N = 1; Eq. 1 / Fig. 1: one B x B similarity matrix serves both directions, text -> image is
// its transpose).  z2_ij = s2 <I_i, T_j> is computed once and kept as ONE matrix of numerators against ONE reference r,
//   E_ij = exp2(z2_ij - r),      r = max(max_i z2_ii, s2 max|I_i| max|T_j| - headroom),
// whose row sums normalise image -> text (beta^A_i) and whose column sums normalise text -> image (beta^C_j).  A
// second pass turns it in place into the combined gradient matrix G_ij = E_ij (beta^A_i + beta^C_j) = P^A_ij + P^C_ji
// (bf16, label entries kept apart in fp32 as before), so that each feature gradient is one contraction:
//   gT = cs G^T I,   gI = cs G T     ->   2 + 4 = 6 B^2 d flop instead of 12.
// One reference for all rows and columns needs every row's and column's largest logit within about 60 (base 2)
// of r + 0; where a total falls under the floor, k_row_merge raises the flag at `gate`, the remaining kernels of
// this path return at once and the two-block path, launched behind them and gated the other way, does the call.

// r of the comment above, and the hand-over flag cleared.  One workgroup.
__global__ __launch_bounds__(1024) void k_sym_ref(const float* zd2, const float* xnorm, const float* ynorm, int64_t B, float s2, float* rglobal,
                                                   int* gate) {
  __shared__ float red[3][16];
  float m[3] = {-INFINITY, 0.f, 0.f};
  const float* src[3] = {zd2, xnorm, ynorm};
  for (int64_t i0 = threadIdx.x; i0 < B; i0 += 4096) {                 // four loads of each array in flight
    float v[3][4];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[a][u] = src[a][i0 + u * 1024 < B ? i0 + u * 1024 : i0];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int u = 0; u < 4; ++u) m[a] = fmaxf(m[a], v[a][u]);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    for (int o = 32; o > 0; o >>= 1) m[a] = fmaxf(m[a], __shfl_xor(m[a], o));
    if ((threadIdx.x & 63) == 0) red[a][threadIdx.x >> 6] = m[a];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
      for (int w = 0; w < 16; ++w) m[a] = fmaxf(m[a], red[a][w]);
    *rglobal = fmaxf(m[0], fmaf(fabsf(s2) * m[1], m[2], -REF_HEADROOM));
    *gate = 0;
  }
}

// One step of sums_over_rows: of the 2 N values per lane a lane keeps the lower or the upper N and adds its partner's, who keeps
// the others.
template <int CTRL, int N>
__device__ __forceinline__ void halve_values(const float (&v)[2 * N], bool upper, float (&out)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const float keep = upper ? v[N + k] : v[k], give = upper ? v[k] : v[N + k];
    out[k] = keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), CTRL, 0xf, 0xf, true));
  }
}
// Sums of col[fm][r] over the 16 lanes of a row (the 16 query rows of a fragment): lane l receives those of fm = l / 2 % 8,
// r = 2 (l % 2) and the next one.  Four steps of half the values each (90 instructions for 32 values), partners l and 15 - l, 7 - l
// of a half row, l ^ 2, l ^ 1.
__device__ __forceinline__ f32x2 sums_over_rows(const float (&col)[8][4], int lane) {
  float v[32], a[16], c[8], e[4], o[2];
#pragma unroll
  for (int k = 0; k < 32; ++k) v[k] = col[k >> 2][k & 3];
  halve_values<0x140>(v, (lane & 8) != 0, a);
  halve_values<0x141>(a, (lane & 4) != 0, c);
  halve_values<0x4E>(c, (lane & 2) != 0, e);
  halve_values<0xB1>(e, (lane & 1) != 0, o);
  return f32x2{o[0], o[1]};
}

// Logit tiles of the symmetric path: k_logit_tiles for one block (X = I on the tile's N side, Y = T on its M side)
// with the one reference; row sums and column sums (over the tile's query rows) come from the accumulators, the latter
// over a lane's four rows, then over the 16 lanes that hold a fragment's rows (sums_over_rows); the four waves that share the
// columns leave their sums in ring unit 4 and, after a barrier, 256 threads add the four.  (So the text -> image normalisation is that
// of the stored, rounded numerators: where a few of them hold a column's mass, their rounding cancels in the gradient.  With the
// unrounded ones gT was 24 % further off at B = 12000, d = 128, 10 % near-duplicate rows.)
// bl.z[0]: E, row partial sums, label numerators; bl.z[1].lpart: column partial sums, one per query tile, cpart[it][j].
// B: the batch rounded up to whole tiles.  RAGGED: the batch is not whole tiles: the
// last key tiles leave their padding columns out (so every row sum is right) and the column sums leave the padding
// rows out; what the padding rows hold in E meets zero feature rows in both contractions.  The loads' bounds spill three more registers there (B = 30000,
// d = 512 1088 -> 1134 us), which the copies that they replace cost more than: us a call 3338 -> 3325, 6145, 320 252 -> 243, 16000, 768 1419 -> 1368, 10241, 128 385 -> 379.
template <bool RAGGED>
__global__ __launch_bounds__(NTHREADS) void k_sym_logit(Blocks bl, int64_t B, int64_t d, float s2, const float* rglobal, int sbi, int sbj) {
  if (gated_off(bl)) return;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const BlockPtrs& p = bl.z[0];
  const int nI = (int)(B / BN), nJ = (int)(B / BM);
  const int total = nI * nJ;
  const int chunk = (total + 7) >> 3, padded = chunk << 3;
  const float ref = *rglobal;
  const float ref2[4] = {ref, ref, ref, ref};
  float* colpart = reinterpret_cast<float*>(smem + 4 * Cfg<256>::UNIT_BYTES);       // [4 waves][256 keys]
  for (int u = blockIdx.x; u < padded; u += gridDim.x) {
    const int lin = (u & 7) * chunk + (u >> 3);
    if ((u >> 3) >= chunk || lin >= total) continue;
    int it, jt;
    superblock_tile(lin, nI, nJ, sbi, sbj, it, jt);
    const int64_t i0 = (int64_t)it * BN, j0 = (int64_t)jt * BM;
    Acc<Cfg<256>::NFA> acc;
#pragma unroll
    for (int i = 0; i < Cfg<256>::NFA; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (RAGGED)
      mainloop<256, FMT_K, FMT_K, true, false, Planes<1, 1>, Bounded>(p.Y + j0 * d, d, p.X + i0 * d, d, (int)(d / BK), smem, acc, 256, 0, 0,
                                                                      Bounded{rows_there<256>(bl.keys - j0), rows_there<256>(bl.rows - i0), 0u});
    else mainloop<256, FMT_K, FMT_K, true>(p.Y + j0 * d, d, p.X + i0 * d, d, (int)(d / BK), smem, acc);
    // the label of query row i is key row i: only the tiles on the diagonal contain label columns
    // (ordinary stores: the matrix is read again by the combining pass and the two contractions)
    // (and of a ragged batch the last key tiles and the last query tiles contain padding)
    float col[Cfg<256>::NFA][4];
    if (it == jt || (RAGGED && (j0 + BM > bl.keys || i0 + BN > bl.rows)))
      logit_epilogue<256, true, true, RAGGED ? MASK_EDGE : MASK_DIAG, false, true>(p, acc, B, s2, i0, j0, 0, LOSS_CLIP, bl.keys, ref2, j0, B, col, bl.rows);
    else logit_epilogue<256, true, true, MASK_NONE, false, true>(p, acc, B, s2, i0, j0, 0, LOSS_CLIP, bl.keys, ref2, j0, B, col);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const f32x2 sums = sums_over_rows(col, lane);
    *reinterpret_cast<f32x2*>(colpart + (wave % 4) * 256 + (wave / 4) * 128 + (lane >> 1 & 7) * 16 + (lane >> 4) * 4 + (lane & 1) * 2) = sums;
    lds_barrier();
    if (t < BM) bl.z[1].lpart[(int64_t)it * B + j0 + t] = (colpart[t] + colpart[256 + t]) + (colpart[512 + t] + colpart[768 + t]);
  }
}

// G_ij = E_ij (beta^A_i + beta^C_j) in place, bf16 (nearest even); the label entries stay 0.  A workgroup takes
// 64 x 64 blocks of the matrix (8 KiB contiguous, see e_index) one after the other; a thread 2 atoms of a block.
__global__ __launch_bounds__(256) void k_sym_combine(Blocks bl, int64_t B) {
  if (gated_off(bl)) return;
  const float* betaA = bl.z[0].beta;
  const float* betaC = bl.z[1].beta;
  uint16_t* E = bl.z[0].E;
  const int64_t nb = B >> 6, nblocks = nb * nb;
  const int t = threadIdx.x;
  for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const int64_t ib = blk / nb, jb = blk % nb;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = h * 256 + t;                          // atom of the block: key piece c >> 6, row c & 63
      const int row = c & 63, col = (c >> 6) * 8;
      u32x4* ptr = reinterpret_cast<u32x4*>(E + blk * 4096 + c * 8);
      const u32x4 raw = *ptr;
      const float ba = betaA[ib * 64 + row];
      const bool padding = ib * 64 + row >= bl.rows;      // a padding row of a ragged batch: exact zeros, whatever it holds
      const f32x4 bc0 = *reinterpret_cast<const f32x4*>(betaC + jb * 64 + col);
      const f32x4 bc1 = *reinterpret_cast<const f32x4*>(betaC + jb * 64 + col + 4);
      const float bc[8] = {bc0[0], bc0[1], bc0[2], bc0[3], bc1[0], bc1[1], bc1[2], bc1[3]};
      u32x4 out;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const __bf16 lo = (__bf16)(bf16_lo(raw[w]) * (ba + bc[2 * w]));
        const __bf16 hi = (__bf16)(bf16_hi(raw[w]) * (ba + bc[2 * w + 1]));
        out[w] = padding ? 0u : (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
      }
      *ptr = out;
    }
  }
}

// Row i of both gradients, for the symmetric path (every row is an own row): with u = sum_ks part[ks][i] = (G T)_i
// without the label entry and gd = (P^A_ii - 1) + (P^C_ii - 1),
//   gI[i] (+)= cs (u + gd T[i])      gT[i] += cs gd I[i]   (the key-side contraction has written or added its part)
// and the row's share of d/ds, <u + gd T[i], I[i]> (sum_ij G_ij S_ij = <G T, I> with the label entries included).
// B: the rows that exist; Bp: row pitch of the partial products.
__global__ __launch_bounds__(256) void k_sym_finalize(Blocks bl, int64_t B, int64_t Bp, int64_t d, float cs, int splitk, int accumulate) {
  if (gated_off(bl)) return;
  const BlockPtrs& p = bl.z[0];
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= B) return;
  const float gd = p.gdiag[i] + bl.z[1].gdiag[i];
  float dot = 0.f;
  for (int64_t k = lane * 4; k < d; k += 256) {
    const u32x2 iw = *reinterpret_cast<const u32x2*>(p.X + i * d + k);
    const u32x2 tw = *reinterpret_cast<const u32x2*>(p.Y + i * d + k);
    const float iv[4] = {bf16_lo(iw[0]), bf16_hi(iw[0]), bf16_lo(iw[1]), bf16_hi(iw[1])};
    const float tv[4] = {bf16_lo(tw[0]), bf16_hi(tw[0]), bf16_lo(tw[1]), bf16_hi(tw[1])};
    f32x4 gi = {0.f, 0.f, 0.f, 0.f};
    if (accumulate) gi = *reinterpret_cast<const f32x4*>(p.gq + i * d + k);
    f32x4 gt = *reinterpret_cast<const f32x4*>(p.gk + i * d + k), u[1];
    sum_slices<1>({p.part + i * d + k}, Bp * d, 0, 1, splitk, u);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ga = fmaf(gd, tv[e], u[0][e]);
      gi[e] = fmaf(cs, ga, gi[e]);
      gt[e] = fmaf(cs * gd, iv[e], gt[e]);
      dot = fmaf(ga, iv[e], dot);
    }
    *reinterpret_cast<f32x4*>(p.gq + i * d + k) = gi;
    *reinterpret_cast<f32x4*>(p.gk + i * d + k) = gt;
  }
  dot = wave_sum(dot);
  if (lane == 0) { p.rowds[i] = dot; bl.z[1].rowds[i] = 0.f; }
}

constexpr int NROWARRAYS = 6;

struct Plan {
  int64_t b, B, d;       // rows taken at a time and B, rounded up to whole tiles: what the tile kernels and the layout below see
  int64_t b_all;         // the share rounded up to whole tiles (b, except where the fused path takes it in chunks)
  bool chunked;          // fused path: rows in chunks, each against all keys, instead of key panels
  int64_t b_real, B_real;
  bool ragged;           // b or B was rounded up
  int64_t W;             // key panel width (B for the materialized path)
  int npanels;
  int tl, tg;            // tile size of the logit kernels and of the gradient kernel (256 or 128)
  int nparts;            // partial row sums per row: one per tl / 2 keys
  int nMq, nMk, nN;      // gradient tiles: query rows, key rows of a panel, columns
  int splitk, ktps;      // query-side split, K-steps per split
  int key_splits, key_ktps;
  size_t off_E, off_lpart, off_rows, off_Xs, off_part, off_kpart, off_ref, total;
  size_t rows_stride;    // bytes of one b-float row array (aligned)
  double us;             // estimated time of the tile kernels
};

// Key panels of the fused path: at most 16384 keys wide (so that one panel of both blocks' numerators
// stays within the 256 MiB last-level cache at the paper's rank shares) and at least two of them.
int fused_panels(int64_t B, int unit) {
  for (int n = 2; n <= 4096; ++n)
    if (B % ((int64_t)n * unit) == 0 && B / n <= 16384) return n;
  return 1;
}

void layout(Plan& pl) {
  const int64_t b = pl.b, B = pl.B, d = pl.d;
  size_t o = 0;
  pl.off_E = o;      o += 2 * align_up((size_t)b * pl.W * 2);
  pl.off_lpart = o;  o += 2 * align_up((size_t)pl.nparts * b * 4);
  pl.rows_stride = align_up((size_t)pl.b_all * 4);
  pl.off_rows = o;   o += 2 * NROWARRAYS * pl.rows_stride;   // ediag, zd2, beta, gdiag, ce, rowds
  pl.off_Xs = o;     o += 2 * align_up((size_t)d * b * 2);
  pl.off_part = o;   o += 2 * align_up((size_t)pl.splitk * b * d * 4);
  pl.off_kpart = o;
  if (pl.key_splits > 1) o += 2 * align_up((size_t)pl.key_splits * B * d * 4);
  pl.off_ref = o;    o += 2 * pl.rows_stride;                            // exponent references of the rows
  // Not used: what a ragged share's padded operands would take.  The sizes that callers ask for, and with them which calls and plans fit
  // a given memory, count it as they always have.
  if (pl.ragged) o += 2 * align_up((size_t)B * d * 2) + 2 * align_up((size_t)pl.b_all * d * 2);
  pl.total = o;
}

// b and B rounded to whole tiles of the two tile sizes, and what follows from them.
void round_shape(Plan& pl, bool fused) {
  const int unit = pl.tl > pl.tg ? pl.tl : pl.tg;
  pl.b = pl.b_all = (pl.b_real + unit - 1) / unit * unit;
  pl.chunked = false;
  pl.B = (pl.B_real + unit - 1) / unit * unit;
  pl.ragged = pl.b_all != pl.b_real || pl.B != pl.B_real;
  pl.npanels = fused ? fused_panels(pl.B, unit) : 1;
  pl.W = pl.B / pl.npanels;
  pl.nparts = (int)(pl.B / (pl.tl / 2));
  pl.nMq = (int)(pl.b / pl.tg);
  pl.nMk = (int)(pl.W / pl.tg);
  pl.nN = (int)((pl.d + pl.tg - 1) / pl.tg);
}

// Widest key panel the fused path may take: half the keys, at most 16384.
int64_t panel_limit(const Plan& pl) {
  const int unit = pl.tl > pl.tg ? pl.tl : pl.tg;
  const int64_t half = (pl.B / unit + 1) / 2 * unit;
  return half < 16384 ? half : 16384;
}

// The fused path's rows in chunks of as many numerators as the widest panel of all rows would hold: logits once instead of
// twice, but the key-side gradient is read and written again per chunk.  Any number of tiles can be cut so, while panels need
// one that divides the keys' tiles (B = 20000 is 79 tiles of 256: 79 panels, 1680 us at N = 20, d = 128, against 170 in
// chunks).  shrink: take that many times smaller chunks.  False where a chunk would be less than a tile.
bool round_to_chunks(Plan& pl, int shrink) {
  const int unit = pl.tl > pl.tg ? pl.tl : pl.tg;
  const int64_t most = pl.b_all * panel_limit(pl) / pl.B / unit / shrink;     // tiles
  if (most == 0) return false;
  const int64_t tiles = pl.b_all / unit, chunks = (tiles + most - 1) / most;
  pl.b = (tiles + chunks - 1) / chunks * unit;
  pl.chunked = true;
  pl.npanels = 1;
  pl.W = pl.B;
  pl.nMq = (int)(pl.b / pl.tg);
  pl.nMk = (int)(pl.W / pl.tg);
  return true;
}

double logits_us(const Plan& pl, int nblk) {
  const double slots = pl.tl == 256 ? CHIP_CUS : 2 * CHIP_CUS, tiles = (double)nblk * (pl.b / pl.tl) * (pl.B / pl.tl);
  const double tile = (double)(pl.d / BK) * step_us(pl.tl, tiles) + (pl.tl == 256 ? 5.5 : 2.5);
  const double rounds = (double)(int64_t)((tiles + slots - 1) / slots), bytes = 2.0 * nblk * pl.b * pl.B;
  return rounds * tile > bytes / BYTES_PER_US ? rounds * tile : bytes / BYTES_PER_US;
}

// the gradient kernel with sk and ks splits, and the finalize kernel's share of reading them back
double grads_us(const Plan& pl, int nblk, int ktps, int sk, int kktps, int ks) {
  const double slots = pl.tg == 256 ? CHIP_CUS : 2 * CHIP_CUS, fix = pl.tg == 256 ? 8.0 : 3.0;
  const double nq = (double)nblk * pl.nMq * pl.nN * sk, nk = (double)nblk * pl.nMk * pl.nN * ks, n = nq + nk;
  const double step = step_us(pl.tg, n), lq = ktps * step + fix, lk = kktps * step + fix, longest = lq > lk ? lq : lk;
  const int slices = nblk * sk;                                      // see k_grads: slices that map onto the 8 XCDs share their L2
  const double spread = slices % 8 == 0 || 8 % slices == 0 ? 1.0 : 1.12;
  // query workgroups first, in rounds of `slots`; the slots that the last of these rounds leaves free start on the key side
  const int s0 = (int)slots, rounds = (int)nq / s0, rest = (int)nq % s0;
  int k = (int)nk / s0;                                              // key workgroups one after the other on such a slot
  auto done = [&] { const double late = k - lq / lk; return k * (double)(s0 - rest) + (late > 0 ? (int)late : 0) * (double)rest; };
  while (done() < nk) ++k;
  const double tail = k * lk > (rest ? lq : 0.0) ? k * lk : lq;
  // (a last query round that fills part of the chip overlaps with the key side less well than that: b = 4096, B = 32768,
  // d = 512 takes 946 us with 2 query splits, half a round, and 837 with 4, one round)
  const double compute = spread * (n <= slots ? longest : rounds * lq + (k || rest ? tail : 0.0) + (rest ? 0.3 * lq * (1.0 - rest / slots) : 0.0));
  const double part = 4.0 * nblk * pl.b * pl.d * sk, key = 4.0 * nblk * pl.W * pl.d * ks;
  const double moved = (4.0 * nblk * pl.b * pl.W + key) / BYTES_PER_US;
  const double splits = (2.0 * part + (ks > 1 ? key + key / ks : 0.0)) / BYTES_PER_US;     // partial sums out and back: not hidden
  return (compute > moved ? compute : moved) + splits;
}

void split(int total, int want, int& splits, int& per) {
  per = (total + want - 1) / want;
  splits = (total + per - 1) / per;                                  // those that are not empty
}

// tile: 0, or the size that the caller's kernels are written for.  limit: most bytes the workspace may take (of
// a call without one of its own: B = 24000, N = 16, d = 512 memory-lean takes 1390 us in 64 MiB and 353 in 148); where no plan
// keeps to it the result's total is above it.
Plan compare_plans(int64_t B, int64_t d, int32_t N, bool fused, int nblk, int tile, size_t limit) {
  static const int Q_SPLITS[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32}, K_SPLITS[] = {1, 2, 3, 4, 6, 8};
  Plan best{};
  best.us = 1e300;
  best.total = ~(size_t)0;
  size_t most = limit;
  // form 0: all rows, in one key panel or several; the memory-lean path's others: rows in chunks.  Those take no more memory than
  // the widest panels would, or the little that a call without a workspace of its own may take.
  for (int form = 0; form < (fused ? 4 : 1); ++form) {
    if (form == 1 && limit == NO_LIMIT) {
      most = best.total + (size_t)4 * best.b_all * (panel_limit(best) > best.W ? panel_limit(best) - best.W : 0);
      if (most < DISCO_STATIC_SCRATCH_BYTES) most = DISCO_STATIC_SCRATCH_BYTES;
    }
    for (int tl = 128; tl <= 256; tl += 128)
      for (int tg = 128; tg <= 256; tg += 128) {
        if (tile && (tl != tile || tg != tile)) continue;
        Plan pl;
        pl.B_real = B; pl.b_real = B / N; pl.d = d; pl.tl = tl; pl.tg = tg;
        round_shape(pl, fused);
        if (form > 0 && !round_to_chunks(pl, 1 << (form - 1))) continue;
        const double base = logits_us(pl, nblk) * (fused && !pl.chunked ? 2 : 1), chunks = (double)((pl.b_all + pl.b - 1) / pl.b);
        const int kt_q = (int)(pl.W / BK), kt_k = (int)(pl.b / BK);
        for (int sk : Q_SPLITS) {
          if (sk > kt_q) break;
          split(kt_q, sk, pl.splitk, pl.ktps);
          for (int ks : K_SPLITS) {
            if (ks > 1 && (fused || tile || ks > kt_k)) break;
            split(kt_k, ks, pl.key_splits, pl.key_ktps);
            double us = base + pl.npanels * grads_us(pl, nblk, pl.ktps, pl.splitk, pl.key_ktps, pl.key_splits);
            // a further chunk reads the key-side gradient back and has its own merge and finalize launches
            us = chunks * us + (chunks - 1.0) * (4.0 * nblk * pl.B * d / BYTES_PER_US + 25.0);
            if (us >= best.us) continue;
            layout(pl);
            if (pl.total > most) continue;
            best = pl;
            best.us = us;
          }
        }
      }
  }
  return best;
}

Plan make_plan(int64_t B, int64_t d, int32_t N, bool fused, int nblk, int tile, size_t limit) {
  static thread_local PlanCache<Plan, 7> cache;
  return cache.get({B, d, N, fused, nblk, tile, (int64_t)limit}, [&] { return compare_plans(B, d, N, fused, nblk, tile, limit); });
}

// Query tiles per super-block of the logit tile walk (superblock_tile): the largest power of two <= 8 that divides
// the query tiles where that is at least 4 (or all of them), else up to 8 with a partial last super-block.
int superblock_width(int nI) {
  int sbi = 8;
  while (nI % sbi) sbi >>= 1;
  if (sbi < 4 && sbi < nI) sbi = nI < 8 ? nI : 8;
  return sbi;
}

// Compute units of the current device rounded down to a multiple of 8 (one persistent workgroup each).
int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
  return n / 8 * 8;
}

template <class K>
bool allow_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

// Numerators written past the caches, or kept in them for the gradient kernel?  They stay in the 256 MiB last-level cache
// until that kernel reads them if they fill at most half of it; what the eight L2s (32 MiB) hold would sit dirty in them, and the
// kernel's end writes it back.  That is worth 1 % on average (12 calls each of d = 64 to 1024, streamed over plain: 16 MiB 0.987, 20 MiB 0.984, single
// calls 0.93 to 1.04), and from 24 MiB to 32 the two are equal to within the boxes' differences (1.006, 0.989, 0.992 on one, 1.005 on
// another), so the line lies there.  (Streamed / plain, us a call of d = 512: 16 MiB, B = 4096, N = 4 57.9 / 59.6; 16384, 64 64.5 / 69.1; 24 MiB, 6144, 6
// 76.3 / 76.9; 32 MiB, 8192, 8 85.2 / 85.4; 64 MiB, B = 32768, N = 64: 148 / 139; 128 MiB, B = 32768, N = 32: 247 / 223; 256 MiB, B = 32768, N = 16:
// 394 / 410; 512 MiB: 724 / 742.)
bool streaming_stores(int nblk, int64_t b, int64_t W) {
  const int64_t bytes = 2 * nblk * b * W;
  return bytes < ((int64_t)24 << 20) || bytes > ((int64_t)144 << 20);
}

// Launchers of one tile size.
template <int T>
struct TileKernels {
  static bool raise_lds() {
    return
        allow_lds(k_logit_tiles<T, true, false>, LOGIT_SMEM_BYTES<T>) && allow_lds(k_logit_tiles<T, true, false, true>, LOGIT_SMEM_BYTES<T>) &&
        allow_lds(k_logit_tiles<T, true, true>, LOGIT_SMEM_BYTES<T>) && allow_lds(k_logit_tiles<T, true, true, true>, LOGIT_SMEM_BYTES<T>) &&
        allow_lds(k_logit_tiles<T, false, true>, LOGIT_SMEM_BYTES<T>) && allow_lds(k_logit_tiles<T, false, true, true>, LOGIT_SMEM_BYTES<T>) &&
        allow_lds(k_logit_tiles<T, true, true, false, false>, LOGIT_SMEM_BYTES<T>) && allow_lds(k_logit_tiles<T, true, true, true, false>, LOGIT_SMEM_BYTES<T>) &&
        allow_lds(k_logit_tiles<T, false, true, false, false>, LOGIT_SMEM_BYTES<T>) && allow_lds(k_logit_tiles<T, false, true, true, false>, LOGIT_SMEM_BYTES<T>) &&
        raise_grads<false>() && raise_grads<true>();
  }
  template <bool RAGGED>
  static bool raise_grads() {
    return allow_lds(k_grads<T, KEY_WRITE, false, RAGGED>, GEMM_SMEM_BYTES<T>) && allow_lds(k_grads<T, KEY_ADD, false, RAGGED>, GEMM_SMEM_BYTES<T>) &&
           allow_lds(k_grads<T, KEY_WRITE, true, RAGGED>, GEMM_SMEM_BYTES<T>) && allow_lds(k_grads<T, KEY_ADD, true, RAGGED>, GEMM_SMEM_BYTES<T>) &&
           allow_lds(k_grads<T, KEY_SPLIT, false, RAGGED>, GEMM_SMEM_BYTES<T>);
  }
  // logit tiles of the key panel [jp0, jp0 + W): statistics, stored numerators or both
  static void logits(bool stats, bool store, const Plan& pl, const Blocks& bl, int64_t g0, float s2, int64_t jp0, int64_t W, int cus, hipStream_t st) {
    const int nI = (int)(pl.b / T), nJ = (int)(W / T);
    // super-block shape of the tile walk: sbi query tiles, then as many key tiles as keep it within 32 tiles
    const int sbi = superblock_width(nI), sbj = 32 / sbi < nJ ? 32 / sbi : nJ;
    const int tiles = bl.nblk * ((nI * nJ + 7) / 8 * 8);  // every block, each padded to a multiple of 8
    const int slots = cus * (T == 256 ? 1 : 2);
    const dim3 grid((unsigned)(tiles < slots ? tiles : slots));
    auto go = [&](auto kernel) { kernel<<<grid, Cfg<T>::NTHREADS, LOGIT_SMEM_BYTES<T>, st>>>(bl, pl.b, pl.B_real, pl.d, g0, s2, jp0, W, sbi, sbj, bl.nblk); };
    auto storing = [&](auto streamed, auto plain) {
      if (streaming_stores(bl.nblk, pl.b, W)) go(streamed);
      else go(plain);
    };
    if (!store) {
      if (pl.ragged) go(k_logit_tiles<T, true, false, true>); else go(k_logit_tiles<T, true, false>);
    } else if (stats) {
      if (pl.ragged) storing(k_logit_tiles<T, true, true, true>, k_logit_tiles<T, true, true, true, false>);
      else storing(k_logit_tiles<T, true, true>, k_logit_tiles<T, true, true, false, false>);
    } else {
      if (pl.ragged) storing(k_logit_tiles<T, false, true, true>, k_logit_tiles<T, false, true, true, false>);
      else storing(k_logit_tiles<T, false, true>, k_logit_tiles<T, false, true, false, false>);
    }
  }
  // both gradient contractions over the key panel [jp0, jp0 + W); part: 0 both, 1 key side only, 2 query side only
  static void grads(int part, bool key_add, bool query_add, const Plan& pl, const Blocks& bl, float cs, int64_t jp0, hipStream_t st) {
    GradShape g;
    g.b = pl.b; g.B = pl.B; g.d = pl.d; g.jp0 = jp0; g.W = pl.W;
    g.nMq = pl.nMq; g.nMk = pl.nMk; g.nN = pl.nN;
    g.splitk = pl.splitk; g.ktps = pl.ktps; g.key_splits = pl.key_splits; g.key_ktps = pl.key_ktps;
    const int qT = pl.nMq * pl.nN, qS = bl.nblk * pl.splitk;
    g.q_wgs = part == 1 ? 0 : qS % 8 == 0 ? qT * qS : 8 % qS == 0 ? 8 * ((qT + 8 / qS - 1) / (8 / qS)) : (qS * qT + 7) / 8 * 8;   // see the kernel's slice -> XCD mapping
    const int k_wgs = part == 2 ? 0 : bl.nblk * ((pl.nMk * pl.nN * pl.key_splits + 7) / 8 * 8);
    auto go = [&](auto kernel) { kernel<<<dim3((unsigned)(g.q_wgs + k_wgs)), Cfg<T>::NTHREADS, GEMM_SMEM_BYTES<T>, st>>>(bl, g, cs); };
    auto instance = [&](auto ragged) {
      constexpr bool R = decltype(ragged)::value;
      if (pl.key_splits > 1) go(k_grads<T, KEY_SPLIT, false, R>);
      else if (query_add) { if (key_add) go(k_grads<T, KEY_ADD, true, R>); else go(k_grads<T, KEY_WRITE, true, R>); }
      else { if (key_add) go(k_grads<T, KEY_ADD, false, R>); else go(k_grads<T, KEY_WRITE, false, R>); }
    };
    if (pl.ragged) instance(std::true_type{});
    else instance(std::false_type{});
  }
};

void finalize(const Problem& pr, const Plan& pl, const Blocks& bl, int64_t g0, float cs, hipStream_t st) {
  FinalizeShape f;
  f.b = bl.rows; f.bp = pl.b; f.B = pl.B_real; f.Bp = pl.B; f.d = pl.d;
  f.g0 = g0; f.splitk = pl.splitk; f.key_splits = pl.key_splits; f.accumulate = pr.accumulate;
  const bool ks = pl.key_splits > 1;
  const int64_t rows = ks ? pl.B_real : bl.rows;
  const bool rowwg = pr.variant != LOSS_NTXENT && rows <= FINALIZE_ROWWG_MAX;
  auto go = [&](auto kernel) { kernel<<<dim3((unsigned)(rowwg ? rows : (rows + 3) / 4)), 256, 0, st>>>(bl, f, cs); };
  if (pr.variant == LOSS_NTXENT) { if (ks) go(k_finalize_ntxent<true>); else go(k_finalize_ntxent<false>); }
  else if (rowwg && !ks && f.d > 256) go(k_finalize<true, false, 2>);
  else if (rowwg) { if (ks) go(k_finalize<true, true, 1>); else go(k_finalize<true, false, 1>); }
  else { if (ks) go(k_finalize<false, true, 1>); else go(k_finalize<false, false, 1>); }
}

// gate / gate_value: see Blocks.  marks: record the benchmark's stage events.
int mfma_run(const Problem& pr, bool fused, const int* gate = nullptr, int gate_value = 0, bool marks = true) {
  const int nblk = loss_blocks(pr.variant);
  const Plan pl = make_plan(pr.B, pr.d, pr.N, fused, nblk, 0, pr.limit);
  const int cus = compute_units();
  const int64_t b = pl.b, ba = pl.b_all, B = pl.B, d = pl.d, W = pl.W;     // whole tiles; the real sizes are pl.b_real, pl.B_real
  char* ws = static_cast<char*>(pr.ws);
  const uint16_t* I = static_cast<const uint16_t*>(pr.I);
  const uint16_t* T = static_cast<const uint16_t*>(pr.T);

  Blocks bl;                                              // all rows of the share

  bl.variant = pr.variant;
  bl.nblk = nblk;
  bl.rows = pl.b_real;
  bl.keys = pl.B_real;
  bl.gate = gate;
  bl.gate_value = gate_value;
  for (int z = 0; z < 2; ++z) {
    BlockPtrs& p = bl.z[z];
    const uint16_t* Xfull = z == 0 ? I : T;
    p.X = Xfull + (size_t)pr.rank * pl.b_real * d;
    p.Y = z == 0 ? T : I;
    p.E = reinterpret_cast<uint16_t*>(ws + pl.off_E + z * align_up((size_t)b * W * 2));
    p.lpart = reinterpret_cast<float*>(ws + pl.off_lpart + z * align_up((size_t)pl.nparts * b * 4));
    char* rows = ws + pl.off_rows + (size_t)z * NROWARRAYS * pl.rows_stride;
    p.ediag = reinterpret_cast<float*>(rows + 0 * pl.rows_stride);
    p.zd2 = reinterpret_cast<float*>(rows + 1 * pl.rows_stride);
    p.beta = reinterpret_cast<float*>(rows + 2 * pl.rows_stride);
    p.gdiag = reinterpret_cast<float*>(rows + 3 * pl.rows_stride);
    p.ce = reinterpret_cast<float*>(rows + 4 * pl.rows_stride);
    p.rowds = reinterpret_cast<float*>(rows + 5 * pl.rows_stride);
    p.ref2 = reinterpret_cast<float*>(ws + pl.off_ref + (size_t)z * pl.rows_stride);
    p.Xs = reinterpret_cast<uint16_t*>(ws + pl.off_Xs + z * align_up((size_t)d * b * 2));
    p.part = reinterpret_cast<float*>(ws + pl.off_part + z * align_up((size_t)pl.splitk * b * d * 4));
    p.kpart = reinterpret_cast<float*>(ws + pl.off_kpart + z * align_up((size_t)pl.key_splits * B * d * 4));
    p.gq = z == 0 ? pr.gI : pr.gT;
    p.gk = z == 0 ? pr.gT : pr.gI;
  }

  const float s2 = pr.s * LOG2E;
  const float c = loss_norm(pl.B_real, pr.variant);
  const float cs = c * pr.s;
  hipStream_t st = pr.stream;
  const bool panels = fused && !pl.chunked;              // statistics first, then the numerators again, panel by panel
  int stage = 0;
  auto mark = [&] { if (marks) stage_mark(st, stage++); };

  mark();
  k_prep<false><<<dim3((unsigned)(nblk * ((ba + 3) / 4))), 256, 0, st>>>(bl, pl.B_real, pl.b_real, ba, d, pr.rank, s2);
  mark();
  for (int64_t r0 = 0; r0 < ba; r0 += b) {                // (one chunk except on the fused path)
    Plan pc = pl;
    pc.b = ba - r0 < b ? ba - r0 : b;
    pc.nMq = (int)(pc.b / pc.tg);
    if (pl.chunked) pc.key_ktps = (int)(pc.b / BK);
    Blocks bc = bl;
    bc.rows = pl.b_real - r0 < pc.b ? pl.b_real - r0 : pc.b;
    for (int z = 0; z < 2; ++z) {
      BlockPtrs& p = bc.z[z];
      p.X += r0 * d;
      p.ediag += r0; p.zd2 += r0; p.beta += r0; p.gdiag += r0; p.ce += r0; p.rowds += r0; p.ref2 += r0;
    }
    const int64_t g0 = (int64_t)pr.rank * pl.b_real + r0;  // global row of the chunk's first row
    const bool key_add = pr.accumulate || r0 > 0;
    auto mark_first = [&] { if (r0 == 0) mark(); };
    if (pl.tl == 256) TileKernels<256>::logits(true, !panels, pc, bc, g0, s2, 0, B, cus, st);
    else TileKernels<128>::logits(true, !panels, pc, bc, g0, s2, 0, B, cus, st);
    mark_first();
    MergeShape mg;
    mg.b = pc.b; mg.Bp = B; mg.d = d; mg.g0 = g0;
    mg.nparts0 = mg.nparts1 = pl.nparts;
    mg.store = !panels; mg.s2 = s2;
    mg.global_ref = nullptr; mg.bad_flag = nullptr;
    mg.fchunks = 1;
    while (mg.fchunks * 2 * nblk * (pc.b / 64) <= cus / 2 && mg.fchunks * 128 <= d) mg.fchunks *= 2;
    k_row_merge<<<dim3((unsigned)(pc.b / 64), (unsigned)nblk, (unsigned)mg.fchunks), 1024, 0, st>>>(bc, mg);
    mark_first();
    for (int pnl = 0; pnl < pl.npanels; ++pnl) {
      const int64_t jp0 = (int64_t)pnl * W;
      if (panels) {
        if (pl.tl == 256) TileKernels<256>::logits(false, true, pc, bc, g0, s2, jp0, W, cus, st);
        else TileKernels<128>::logits(false, true, pc, bc, g0, s2, jp0, W, cus, st);
      }
      auto grads = [&](int part) {
        if (pl.tg == 256) TileKernels<256>::grads(part, key_add, pnl > 0, pc, bc, cs, jp0, st);
        else TileKernels<128>::grads(part, key_add, pnl > 0, pc, bc, cs, jp0, st);
      };
      if (fused || !marks || !stage_marks_on()) {
        grads(0);
      } else {                                            // a launch of its own for each side, so that each can be timed
        grads(1);
        mark();
        grads(2);
      }
    }
    if (!fused && !stage_marks_on()) ++stage;
    if (r0 + b >= ba) mark();
    finalize(pr, pc, bc, g0, cs, st);
  }
  k_scalars<<<1, 1024, 0, st>>>(bl, pl.b_real, c, pr.accumulate, pr.loss, pr.gs);
  mark();
  return hipGetLastError() == hipSuccess ? DISCO_OK : DISCO_ERR_HIP;
}

// The symmetric full loss (see the kernels above): one matrix of numerators, both directions' statistics, one
// combined gradient matrix, two contractions; then, behind the flag, the two-block path for inputs it cannot take.
// A small batch is not worth the path's two fixed costs, the pass over the matrix that combines the gradients and the
// empty launches of the two-block path behind it (about 45 us together): the 6 B^2 d flop it saves pay for them from about
// B^2 d = 1e10 on.  (Measured, symmetric / two-block in us: B = 2816, d = 640: 128 / 102; 4375, 320: 182 / 146;
// 3964, 256: 149 / 99; 6912, 320: 239 / 255; 8728, 320: 344 / 470.)
bool sym_two_block(int64_t B, int64_t d) { return (double)B * B * d < 1e10; }

// Behind the larger of the two plans' workspaces: the hand-over flag and the reference.
constexpr size_t SYM_WORDS = 256;
size_t sym_plan_limit(size_t limit) { return limit == NO_LIMIT ? NO_LIMIT : limit - SYM_WORDS; }
size_t sym_tail(int64_t B, int64_t d, size_t limit) {
  const size_t a = make_plan(B, d, 1, false, 1, 256, sym_plan_limit(limit)).total, c = make_plan(B, d, 1, false, 2, 0, sym_plan_limit(limit)).total;
  return a > c ? a : c;
}

int mfma_sym_run_impl(const Problem& pr) {
  if (sym_two_block(pr.B, pr.d)) {
    const int status = mfma_run(pr, false);
    stage_mark(pr.stream, DISCO_STAGES_SYMMETRIC);
    return status;
  }
  const Plan pl = make_plan(pr.B, pr.d, 1, false, 1, 256, sym_plan_limit(pr.limit));
  const int persistent_wgs = compute_units();
  const int64_t B = pl.B, d = pl.d, Br = pl.B_real;        // whole tiles / the rows that exist
  char* ws = static_cast<char*>(pr.ws);
  const size_t tail = sym_tail(Br, d, pr.limit);
  int* gate = reinterpret_cast<int*>(ws + tail);
  float* rglobal = reinterpret_cast<float*>(ws + tail + 128);
  const uint16_t* I = static_cast<const uint16_t*>(pr.I);
  const uint16_t* T = static_cast<const uint16_t*>(pr.T);

  Blocks bl;
  bl.variant = LOSS_CLIP;
  bl.nblk = 1;
  bl.rows = Br;
  bl.keys = Br;
  bl.gate = nullptr;
  bl.gate_value = 0;
  BlockPtrs& p = bl.z[0];
  char* rows0 = ws + pl.off_rows;
  char* rows1 = rows0 + (size_t)NROWARRAYS * pl.rows_stride;
  p.X = I;
  p.Y = T;
  p.E = reinterpret_cast<uint16_t*>(ws + pl.off_E);
  p.lpart = reinterpret_cast<float*>(ws + pl.off_lpart);
  p.ediag = reinterpret_cast<float*>(rows0 + 0 * pl.rows_stride);
  p.zd2 = reinterpret_cast<float*>(rows0 + 1 * pl.rows_stride);
  p.beta = reinterpret_cast<float*>(rows0 + 2 * pl.rows_stride);
  p.gdiag = reinterpret_cast<float*>(rows0 + 3 * pl.rows_stride);
  p.ce = reinterpret_cast<float*>(rows0 + 4 * pl.rows_stride);
  p.rowds = reinterpret_cast<float*>(rows0 + 5 * pl.rows_stride);
  p.ref2 = reinterpret_cast<float*>(ws + pl.off_ref);
  p.Xs = reinterpret_cast<uint16_t*>(ws + pl.off_Xs);
  p.part = reinterpret_cast<float*>(ws + pl.off_part);
  p.gq = pr.gI;
  p.gk = pr.gT;
  // "block 1" holds the column side: partial column sums and the text -> image statistics; label numerators,
  // positive-pair logits and the reference are the row side's
  BlockPtrs& q = bl.z[1];
  q = p;
  q.lpart = reinterpret_cast<float*>(ws + pl.off_lpart + align_up((size_t)pl.nparts * B * 4));
  q.beta = reinterpret_cast<float*>(rows1 + 2 * pl.rows_stride);
  q.gdiag = reinterpret_cast<float*>(rows1 + 3 * pl.rows_stride);
  q.ce = reinterpret_cast<float*>(rows1 + 4 * pl.rows_stride);
  q.rowds = reinterpret_cast<float*>(rows1 + 5 * pl.rows_stride);
  q.ref2 = reinterpret_cast<float*>(ws + pl.off_ref + pl.rows_stride);

  const float s2 = pr.s * LOG2E;
  const float c = loss_norm(Br, LOSS_CLIP);
  const float cs = c * pr.s;
  hipStream_t st = pr.stream;
  const int nT = (int)(B / BN);
  const int sbi = superblock_width(nT);
  const int sbj = 32 / sbi < nT ? 32 / sbi : nT;
  const int tiles = (nT * nT + 7) / 8 * 8;
  const dim3 logit_grid((unsigned)(tiles < persistent_wgs ? tiles : persistent_wgs));
  int stage = 0;

  stage_mark(st, stage++);
  k_prep<true><<<dim3((unsigned)((B + 3) / 4)), 256, 0, st>>>(bl, Br, Br, B, d, 0, s2);
  k_sym_ref<<<1, 1024, 0, st>>>(p.zd2, p.beta, p.gdiag, Br, s2, rglobal, gate);
  stage_mark(st, stage++);
  if (pl.ragged) k_sym_logit<true><<<logit_grid, NTHREADS, LOGIT_SMEM_BYTES<256>, st>>>(bl, B, d, s2, rglobal, sbi, sbj);
  else k_sym_logit<false><<<logit_grid, NTHREADS, LOGIT_SMEM_BYTES<256>, st>>>(bl, B, d, s2, rglobal, sbi, sbj);
  stage_mark(st, stage++);
  Blocks both = bl;
  both.nblk = 2;
  MergeShape mg;
  mg.b = B; mg.Bp = B; mg.d = d; mg.g0 = 0;
  mg.nparts0 = pl.nparts; mg.nparts1 = nT;
  mg.store = 0; mg.fchunks = 0; mg.s2 = s2;
  mg.global_ref = rglobal; mg.bad_flag = gate;
  k_row_merge<<<dim3((unsigned)(B / 64), 2), 1024, 0, st>>>(both, mg);
  Blocks go = bl;                                   // from here on only while no total was lost
  go.gate = gate;
  go.gate_value = 0;
  k_transpose<<<dim3((unsigned)(B / 64)), 1024, 0, st>>>(go, B, d);
  stage_mark(st, stage++);
  k_sym_combine<<<dim3((unsigned)(8 * persistent_wgs)), 256, 0, st>>>(go, B);
  stage_mark(st, stage++);
  auto grads = [&](int part) { TileKernels<256>::grads(part, pr.accumulate != 0, false, pl, go, cs, 0, st); };
  if (stage_marks_on()) {
    grads(1);
    stage_mark(st, stage++);
    grads(2);
  } else {
    grads(0);
    ++stage;
  }
  stage_mark(st, stage++);
  stage_mark(st, stage++);
  k_sym_finalize<<<dim3((unsigned)((Br + 3) / 4)), 256, 0, st>>>(go, Br, B, d, cs, pl.splitk, pr.accumulate);
  Blocks go2 = go;
  go2.nblk = 2;
  k_scalars<<<1, 1024, 0, st>>>(go2, Br, c, pr.accumulate, pr.loss, pr.gs);
  stage_mark(st, stage++);
  if (hipGetLastError() != hipSuccess) return DISCO_ERR_HIP;
  Problem two_block = pr;
  two_block.limit = sym_plan_limit(pr.limit);
  return mfma_run(two_block, false, gate, 1, false);
}

}  // namespace

bool mfma_supported(int64_t B, int64_t d, int32_t N, int dtype, int variant) {
  if (dtype != DISCO_BF16) return false;
  if (N <= 0 || B % N != 0) return false;
  const int64_t b = B / N;
  if (variant == LOSS_NTXENT && B % 2 != 0) return false;                   // two views
  // per-lane load offsets are 32-bit byte offsets inside one operand tile: 256 rows of pitch b (Xs) or four block
  // rows of pitch 64 W (row groups of the stored numerators) must stay below 4 GiB
  if (B > ((int64_t)1 << 23) || b > ((int64_t)1 << 22)) return false;      // (rounding up to whole tiles stays within them)
  return d % 64 == 0;
}

bool mfma_whole_tiles(int64_t B, int32_t N) { return N > 0 && B % N == 0 && (B / N) % 256 == 0; }

double mfma_stored_estimate_us(int64_t B, int64_t d, int32_t N, int variant) { return make_plan(B, d, N, false, loss_blocks(variant), 0, NO_LIMIT).us; }
size_t mfma_workspace_bytes(int64_t B, int64_t d, int32_t N, int variant, bool fused, size_t limit) {
  return make_plan(B, d, N, fused, loss_blocks(variant), 0, limit).total;
}
bool mfma_raise_lds() {
  return TileKernels<256>::raise_lds() && TileKernels<128>::raise_lds() && allow_lds(k_sym_logit<false>, LOGIT_SMEM_BYTES<256>) &&
         allow_lds(k_sym_logit<true>, LOGIT_SMEM_BYTES<256>);
}
int mfma_stored_run(const Problem& pr) { return mfma_run(pr, false); }
int mfma_fused_run(const Problem& pr) { return mfma_run(pr, true); }
size_t mfma_sym_workspace_bytes(int64_t B, int64_t d, size_t limit) {
  if (sym_two_block(B, d)) return make_plan(B, d, 1, false, 2, 0, limit).total;
  const size_t tail = sym_tail(B, d, limit);
  return tail == NO_LIMIT ? tail : tail + SYM_WORDS;
}
int mfma_sym_run(const Problem& pr) { return mfma_sym_run_impl(pr); }

void mfma_describe(int64_t B, int64_t d, int32_t N, int variant, bool fused, bool sym, size_t limit, disco_plan* out) {
  const bool one = sym && !sym_two_block(B, d);
  const Plan pl = one ? make_plan(B, d, 1, false, 1, 256, sym_plan_limit(limit)) : make_plan(B, d, N, fused, loss_blocks(variant), 0, limit);
  out->kernels = one ? DISCO_KERNELS_SYMMETRIC : DISCO_KERNELS_TILES;
  if (pl.total == NO_LIMIT) return;
  out->logit_tile = pl.tl;
  out->gradient_tile = pl.tg;
  out->row_chunks = (int)((pl.b_all + pl.b - 1) / pl.b);
  out->key_panels = pl.npanels;
  out->query_splits = pl.splitk;
  out->key_splits = pl.key_splits;
  out->microseconds = pl.us;
}

}  // namespace disco

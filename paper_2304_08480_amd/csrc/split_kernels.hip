// The fp32 path's large calls: its four contractions on the 16-bit matrix instructions, with every fp32 operand split into planes
// whose products are exact in the instruction and summed in fp32.  Two forms:
//   fp16   two planes of 11 significand bits each.  A logit is four plane products, a gradient entry three (bf16 features, one plane: one
//          and two).  What the planes leave out of a value is 0 three times in four, else 2^-24 to 2^-23 of it; the product left out of a gradient is
//          2^-24.6 (root mean square).  fp16's range is what features have to keep to (k_feature_halves tests them on the device).  Rows of
//          gradient entries that it would be too narrow for are multiplied by a power of two of their own (row_shift).
//   bf16   three planes of 8 bits, which add up to the value exactly over nearly all of fp32's range: six plane products (three against bf16
//          features; one between them).  The six leave out 2^-27.5 of a product (root mean square; the worst case is 2^-24).  For
//          features that the fp16 form cannot hold, and for calls too small to gain from it.
// One product over the whole reduction follows the other, the smallest first (SWEEPS), so that only the last one rounds at the size of
// the result: that is what decides the errors where logits are small, and why the fp16 form's are mostly no larger although its planes hold a bit less.
// Against 64 bits, 2-norm of the gradients, fp16 over bf16 planes (logits in sweeps, gradients piece by piece), geometric mean over inputs, unit rows:
//   bf16 features  d = 100 to 1000, s = 1/0.07 to 100, positives of cosine 0.27 to 0.89: 0.72 to 1.02
//   fp32 features  d = 192 to 1024, by cosine 0.89 / 0.64 / 0.38 / 0.27:  s = 1/0.07 0.98 / 0.95 / 0.66 / 0.62;  30 0.99 / 0.98 / 0.96 / 0.84
//                  and where rounding of single logits decides (few rows hold the gradient) 1.0 in the mean, one input 0.2 to 5
// Where a logit is short of terms and multiplied by much, the features' lost bits show: fp32 features, cosine 0.27, s = 50 1.18 at d = 64, 1.1 at 77 and 100, 1.0 at 192;
// s = 100 1.27, 1.2, 1.11, 1.06 at 256 and 320; cosine 0.89, s = 30 1.27 at 64, 1.08 at 100 and 128.  Such calls stay on bf16 planes (halves_planned, halves_hold).
// What is relative to the largest rows is a gradient as a whole: entries and rows of it as far below them as 2^-35 of a row of G (2^-51 of 1 in rows of
// more than 2^-16) keep fewer bits than bf16 planes leave them, and can be 0.  (s = 100, keys of other ranks.)
//
// What bounds the fp32 matrix instruction is its rate, 157 TFLOP/s, of which the products straight from memory
// (naive_kernels.hip) reach 80 and LDS-tiled ones reached 91 (58 % at their largest); six bf16 products at 1.2 PFLOP/s are 200 TFLOP/s
// of fp32 work.  Measured, us a call, bf16 / fp16 planes: fp32 features B = 8192, N = 8, d = 512: 290 / 210, now 204 (logits 68, softmax 28, both
// gradient sides 102); 12288, 4, 256: 806 / 561; 10416, 8, 1024: 1029 / 691; 4096, 16, 512: 83 / 70; bf16 features 12288, 8, 100: 220 / 181;
// 110 drawn fp32 calls: 0.78 in the median, with those of narrow features and large multipliers that halves_hold has since kept on bf16 planes.
//
// Per block (X: the rank's rows, Y: all rows):
//   planes    features -> planes, rows padded with zeros to whole tiles, columns to whole 64-deep K-steps
//   logits    S = X Y^T in fp32 (b x B)
//   softmax   row by row against the row's true maximum: loss terms, G = softmax - onehot as planes (fp16: times the row's own power of two)
//   grads     gY = cs G^T X (key side) and the split-K partial sums of G Y (query side), one launch
//   finalize  partial sums into the gradients, loss and d/ds
// The rows are taken in chunks where the whole would need more memory than the fp32 blocks of the small kernels do.
#include "common.h"
#include "mfma_tile.h"

namespace disco {
namespace {

using namespace tile;

// Written on the device by k_feature_halves, k_feature_planes and the softmax: in which form the call's features and gradient entries are kept.
// At the front of the workspace, where tests read which form a call took.
struct HalfHead {
  uint32_t mark;         // HEAD_MARK: the plan is one for fp16 planes
  uint32_t half;         // 1: fp16 planes, 0: bf16 planes
  float unscale[2];      // what undoes the power of two that the features of I (of T) are multiplied with
  uint32_t shifted;      // some row of G is multiplied by a power of two of its own
};
constexpr uint32_t HEAD_MARK = 0x666c6168u;
constexpr int HALF_FLAGS = 1024;                         // workgroups of k_feature_halves at most, a flag each
constexpr size_t HEAD_BYTES = 8192;                      // head and flags (in 4352, at no multiple of 4 KiB, the arrays behind them cost a call of B = 8192, N = 8, d = 512 0.6 us of 202)
static_assert(sizeof(HalfHead) <= 256 && 256 + HALF_FLAGS * sizeof(uint32_t) <= HEAD_BYTES);
constexpr float G_SCALE = 0x1p15f, REST_SCALE = 0x1p11f; // fp16 planes of a gradient entry: see store_unit_halves
// Rows of G whose largest entry is below 2^-16 are multiplied by the power of two that brings it to [2^-12, 2^-11) (by 2^100 at most: an entry
// of 2^-112, about where bf16 planes end).  Higher up they would keep more of their own small entries, but a row that lies beside undecided ones moves
// that much of its power of two into the features' planes (RowShifts of mfma_tile.h).
constexpr int ROW_LEAST_EXP = -16, ROW_SHIFTED_EXP = -12, ROW_SHIFT_MOST = 100;
constexpr uint8_t NO_ROW = 255;

struct SplitBlock {
  const uint16_t* X;     // planes of the rank's rows: the first of the chunk
  const uint16_t* Y;     // planes of all rows
  float* S;              // bp x Bp logits without the multiplier
  uint16_t* G;           // three (fp16: two) planes, bp x Bp each
  float* part;           // splitk x bp x dp query-side sums
  float* kpart;          // key_splits x Bp x dp key-side sums (only where they do not go straight to gk)
  float* gq;             // query-side destination (the whole B x d matrix)
  float* gk;             // key-side destination
  float* ce;             // b: cross-entropy of the rank's rows
  float* ds;             // b: row shares of d/ds
  uint8_t* shift;        // (fp16) rows of the chunk: the exponent of the row's power of two, 255 for a row of zeros
};
struct SplitArgs {
  SplitBlock z[2];
  int64_t b, bp;         // rows of the chunk and the same rounded up to whole tiles
  int64_t B, Bp;         // all rows, rounded up: also the pitch of S and G
  int64_t d, dp;         // feature width, rounded up to a multiple of 64: the pitch of the planes and of the partial sums
  int64_t g0;            // global row of the chunk's first row
  int64_t r0;            // local row of the chunk's first row
  int64_t fplane, gplane;  // elements between feature planes / between planes of G
  int nb, variant;
  int nMq, nMk, nN;      // gradient tiles: query rows, key rows, columns
  int splitk, ktps, key_splits, key_ktps;  // splits of the two reductions and their length in 64-deep pieces
  int q_wgs;
  HalfHead* head;        // null: bf16 planes
};

// v = p[0] + p[1] + p[2], to the last bit while the last plane stays above the smallest bf16 (a value above about 2^-109).  (A value whose leading plane
// would round to infinity keeps a cut one; a value that is not finite is its own leading plane.)
struct Three { uint16_t p[3]; };
__device__ __forceinline__ uint16_t bf16_bits(float f) {
  const __bf16 v = (__bf16)f;
  return __builtin_bit_cast(uint16_t, v);
}
__device__ __forceinline__ float bf16_value(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ Three split3(float v) {
  Three t;
  t.p[0] = bf16_bits(v);
  const bool over = (t.p[0] & 0x7f80u) == 0x7f80u;                     // not finite, or rounded up to it
  if (over) t.p[0] = (uint16_t)(__float_as_uint(v) >> 16);
  const bool finite = (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u;
  if (over && !finite && v != v) t.p[0] = 0x7fc0u;                     // NaN stays one
  const float r1 = finite ? v - bf16_value(t.p[0]) : 0.f;
  t.p[1] = bf16_bits(r1);
  t.p[2] = bf16_bits(r1 - bf16_value(t.p[1]));
  return t;
}
__device__ __forceinline__ void store_planes(uint16_t* dst, int64_t plane, const f32x4& v) {
  u32x2 w[3];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const Three a = split3(v[2 * h]), c = split3(v[2 * h + 1]);
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q][h] = (uint32_t)a.p[q] | (uint32_t)c.p[q] << 16;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2*>(dst + q * plane) = w[q];
}

// The planes of four values of [-1, 1] or NaN (gradient entries: nothing overflows, NaN makes all three NaN).
__device__ __forceinline__ void store_unit_planes(uint16_t* dst, int64_t plane, const f32x4& v) {
  f32x4 rest = v;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    bf16x4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (__bf16)rest[e];
    const u32x2 w = __builtin_bit_cast(u32x2, h);
    *reinterpret_cast<u32x2*>(dst + q * plane) = w;
#pragma unroll
    for (int e = 0; e < 4; ++e) rest[e] -= __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
  }
}

// The fp16 planes of four gradient entries x m / 2^15 (values of [-1, 1] or NaN): g 2^15 = h + l 2^-11, h and l of 11 significand bits each, so
// that h keeps all of them down to |g| = 2^-29 and l down to 2^-28.  What both leave out of an entry is 2^-51 at most, so rows of nothing larger than 2^-16
// are multiplied up first (row_shift): it is then 2^-35 of a row's largest entry at most.  (x m 2^11 is rounded as x m is, so the fused product-sum below is exact; it
// and the conversion are one instruction.  h passes through an empty asm statement because the compiler would otherwise form the h
// that l is taken from a second time, by an instruction that rounds x m once where the stored one is rounded twice.)
__device__ __forceinline__ void store_unit_halves(uint16_t* dst, int64_t plane, const f32x4& x, float m) {
  const float m2 = m * REST_SCALE;
  half4 h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = (_Float16)(x[e] * m);
  u32x2 w = __builtin_bit_cast(u32x2, h);
  asm("" : "+v"(w));
  h = __builtin_bit_cast(half4, w);
#pragma unroll
  for (int e = 0; e < 4; ++e) l[e] = (_Float16)fmaf((float)h[e], -REST_SCALE, x[e] * m2);
  *reinterpret_cast<u32x2*>(dst) = w;
  *reinterpret_cast<half4*>(dst + plane) = l;
}

// The exponent of the power of two that a row of G is multiplied with, from its largest entry: the label's, off-label mass / total.
__device__ __forceinline__ int row_shift(float top) {
  const int x = (int)(__float_as_uint(top) >> 23) - 127, e = ROW_SHIFTED_EXP - x;
  return !(top > 0.f) || x >= ROW_LEAST_EXP ? 0 : e < ROW_SHIFT_MOST ? e : ROW_SHIFT_MOST;
}
// 2^e, -126 <= e <= 127
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

// Four features from column k on of a row that starts at p, as fp32; 0 from column d on.
template <int DT, bool VEC>
__device__ __forceinline__ f32x4 load_features(const void* src, int64_t at, int64_t k, int64_t d) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (DT == DISCO_BF16) {
    const uint16_t* p = static_cast<const uint16_t*>(src) + at + k;
    if constexpr (VEC) {
      if (k < d) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < d) v[e] = bf16_value(p[e]);
    }
  } else {
    const float* p = static_cast<const float*>(src) + at + k;
    if constexpr (VEC) {
      if (k < d) v = *reinterpret_cast<const f32x4*>(p);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < d) v[e] = p[e];
    }
  }
  return v;
}

// Features as fp16 planes.  A matrix is multiplied with the power of two that brings the largest entry of its first row into [2^10, 2^11);
// an entry x of the product is h + l, 11 significand bits each (bf16 features: h alone), and h 2^-11 is kept as well, the partner
// of the gradient entries' second plane, which is 2^11 times what it stands for.  Beyond the planes' own bits that loses 2^-28 of a row's largest
// entry at most where every entry is under 2^15.9 and every row's largest is 0 or at least 2^3: the planes end at 2^-24.  A workgroup that
// sees anything else (rows whose norms differ by more than 2^5 to 2^7, what is not finite, a first row of zeros) raises its flag, and
// k_feature_planes replaces the planes of the whole call by bf16 ones.  One wave (LPR = 64) or 16 lanes a row.
template <int DT, bool VEC, int LPR>
__global__ __launch_bounds__(256) void k_feature_halves(const void* I, const void* T, int64_t B, int64_t d, int64_t rows, int64_t dp, int mats,
                                                        uint16_t* Ip, uint16_t* Tp, HalfHead* head, uint32_t* flags) {
  __shared__ float first[2][4];
  float m[2] = {0.f, 0.f};
#pragma unroll
  for (int z = 0; z < 2; ++z)
    if (z < mats) {
      for (int64_t k = threadIdx.x * 4; k < d; k += 1024) {
        const f32x4 v = load_features<DT, VEC>(z ? T : I, 0, k, d);
#pragma unroll
        for (int e = 0; e < 4; ++e) m[z] = fmaxf(m[z], fabsf(v[e]));
      }
      m[z] = wave_reduce(m[z], [](float a, float b) { return fmaxf(a, b); });
      if ((threadIdx.x & 63) == 0) first[z][threadIdx.x >> 6] = m[z];
    }
  __syncthreads();
  int e[2] = {0, 0};
  bool bad = false;
#pragma unroll
  for (int z = 0; z < 2; ++z)
    if (z < mats) {
      const float top = fmaxf(fmaxf(first[z][0], first[z][1]), fmaxf(first[z][2], first[z][3]));
      e[z] = 137 - (int)(__float_as_uint(top) >> 23);                // 10 - exponent; the scales below stay far from fp32's ends
      bad = bad || e[z] < -80 || e[z] > 80;
    }
  const int both = e[0] + e[mats - 1];
  bad = bad || both < -120 || both > 120;
  if (bad) e[0] = e[1] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 2) head->unscale[threadIdx.x] = __uint_as_float((uint32_t)(127 - (threadIdx.x ? e[1] : e[0])) << 23);
  const int64_t plane = rows * dp, step = (int64_t)gridDim.x * (256 / LPR);
  const int lane = threadIdx.x % LPR;
  const int64_t todo = bad ? 0 : mats * rows;                         // (a test in the loop, for rows further on, cost the others 1 us of 18)
  for (int64_t w = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR; w < todo; w += step) {
    const bool second = w >= rows;
    const int64_t row = second ? w - rows : w;
    const float scale = __uint_as_float((uint32_t)(127 + (second ? e[1] : e[0])) << 23);
    uint16_t* dst = (second ? Tp : Ip) + row * dp;
    float top = 0.f;
    for (int64_t k = lane * 4; k < dp; k += LPR * 4) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (row < B) v = load_features<DT, VEC>(second ? T : I, row * d, k, d);
      half4 h, l, low;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float x = v[c] * scale, size = fabsf(x);
        bad = bad || !(size < 61000.f);
        top = fmaxf(top, size);
        h[c] = (_Float16)x;
        l[c] = (_Float16)(x - (float)h[c]);
        low[c] = (_Float16)((float)h[c] * (1.f / REST_SCALE));
      }
      *reinterpret_cast<half4*>(dst + k) = h;
      if constexpr (DT == DISCO_F32) *reinterpret_cast<half4*>(dst + plane + k) = l;
      *reinterpret_cast<half4*>(dst + (DT == DISCO_F32 ? 2 : 1) * plane + k) = low;
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    bad = bad || (top > 0.f && top < 8.f);
  }
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) flags[blockIdx.x] = any;
}

// Feature planes of I (z = 0) and T: rows x dp each, zero from row B and from column d on.  VEC: whole 16-byte (bf16: 8-byte)
// pieces of a row can be read at once.  mats: 1 for the two-view loss, whose matrices are one.  Four columns per thread,
// grid-stride.  head: the call's features are fp16 planes unless a flag of k_feature_halves is raised; decides that for the kernels that
// follow, and is done if none is.
template <int DT, bool VEC>
__global__ __launch_bounds__(256) void k_feature_planes(const void* I, const void* T, int64_t B, int64_t d, int64_t rows, int64_t dp,
                                                        int mats, uint16_t* Ip,
                                                        uint16_t* Tp, HalfHead* head, const uint32_t* flags, int nflags) {
  if (head) {
    uint32_t f[HALF_FLAGS / 256];
#pragma unroll
    for (int u = 0; u < HALF_FLAGS / 256; ++u) {
      const int i = threadIdx.x + u * 256;
      f[u] = i < nflags ? flags[i] : 0u;
    }
    uint32_t any = 0u;
#pragma unroll
    for (int u = 0; u < HALF_FLAGS / 256; ++u) any |= f[u];
    const bool half = !__syncthreads_or((int)any);
    if (blockIdx.x == 0 && threadIdx.x == 0) { head->mark = HEAD_MARK; head->half = half; head->shifted = 0u; }
    if (half) return;
  }
  const int64_t cpr = dp >> 2, n = rows * cpr, plane = rows * dp;
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < mats * n; c += (int64_t)gridDim.x * 256) {
    const bool second = c >= n;
    const int64_t w = second ? c - n : c, row = w / cpr, k = (w - row * cpr) * 4;
    const void* src = second ? T : I;
    uint16_t* dst = (second ? Tp : Ip) + row * dp + k;
    if constexpr (DT == DISCO_BF16) {
      u32x2 v = {0u, 0u};
      const uint16_t* p = static_cast<const uint16_t*>(src) + row * d + k;
      if (row < B) {
        if constexpr (VEC) {
          if (k < d) v = *reinterpret_cast<const u32x2*>(p);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < d) v[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
        }
      }
      *reinterpret_cast<u32x2*>(dst) = v;
    } else {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      const float* p = static_cast<const float*>(src) + row * d + k;
      if (row < B) {
        if constexpr (VEC) {
          if (k < d) v = *reinterpret_cast<const f32x4*>(p);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < d) v[e] = p[e];
        }
      }
      store_planes(dst, plane, v);
    }
  }
}

// S = X Y^T, one T x T tile per workgroup (rows: query, columns: key).  NP: planes of a feature (1 or 3).
template <int T, int NP>
__global__ __launch_bounds__(Cfg<T>::NTHREADS) void k_split_logits(SplitArgs a, int sbi, int sbj) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nI = (int)(a.bp / T), nJ = (int)(a.Bp / T), total = nI * nJ, per_block = (total + 7) / 8 * 8;
  const int z = blockIdx.x / per_block;
  int lin, it, jt;
  if (!xcd_linear(blockIdx.x - z * per_block, total, lin)) return;
  superblock_tile(lin, nI, nJ, sbi, sbj, it, jt);
  const SplitBlock& p = a.z[z];
  const int64_t i0 = (int64_t)it * T, j0 = (int64_t)jt * T;
  Acc<Cfg<T>::NFA> acc;
  auto products = [&](auto ps) {
    using PS = decltype(ps);
    mainloop<T, FMT_K, FMT_K, false, true, PS>(p.X + i0 * a.dp, a.dp, p.Y + j0 * a.dp, a.dp, (int)(a.dp / BK) * PS::N, smem, acc, T, a.fplane, a.fplane);
  };
  float scale = 1.0f;
  if (a.head && a.head->half) {
    scale = a.head->unscale[0] * a.head->unscale[a.nb - 1];
    products(HalfLogits<(NP + 1) / 2>{});
  } else {
    products(Planes<NP, NP, NP == 3>{});
  }
  store_tile_f32<T, false>(acc, smem, p.S + i0 * a.Bp + j0, a.Bp, scale);
}

constexpr int SM_THREADS = 512;                          // softmax: threads per row
constexpr int SM_WAVES = SM_THREADS / 64;

// One workgroup per row: maximum over the columns that take part, cross-entropy, the row's share of d/ds and the row of
// G = softmax - onehot as planes (0 in the padding columns and rows, and in a two-view row's own column).  The off-label
// mass is summed on its own, so that P_label - 1 = -(it) / (total) does not cancel, and d/ds as
// sum_{j != label} P_ij (S_ij - S_i,label).  134 MB at B = 8192, N = 8 take 28.5 us, 4.7 TB/s (33 with a product in every step of
// the maximum, 68 registers, five barriers instead of two and eight instructions for a value's planes instead of five): memory and the 26
// vector instructions an element about even.  Pieces that hold no special column take no tests.  KEEP: 4-column pieces a thread keeps, the
// smallest of 4 (Bp <= 8192; 44 registers, so that four workgroups share a compute unit, not three), 8 (16384) and 16 (32768) that holds
// the row, which is then read once; else (0) three times, from cache, with every exponential taken twice (us a call, 0 / 16: B = 32768,
// N = 8, d = 512 4394 / 4225; 20000, 8, 256 1148 / 1095).
template <int KEEP>
__global__ __launch_bounds__(SM_THREADS) void k_split_softmax(SplitArgs a, float s) {
  __shared__ float red[3][SM_WAVES];
  const int64_t i = blockIdx.x;
  const SplitBlock& p = a.z[blockIdx.y];
  uint16_t* G = p.G + i * a.Bp;
  const int64_t nvec = a.Bp >> 2;
  const bool half = a.head && a.head->half;
  if (i >= a.b) {
    for (int64_t q = threadIdx.x; q < nvec; q += SM_THREADS)
      for (int pl = 0; pl < (half ? 2 : 3); ++pl) *reinterpret_cast<u32x2*>(G + pl * a.gplane + q * 4) = u32x2{0u, 0u};
    return;
  }
  const float* S = p.S + i * a.Bp;
  const int64_t label = label_row(a.g0 + i, a.B, a.variant), self = masked_col(a.g0 + i, a.variant);
  const float xl = S[label];
  const int B = (int)a.B, lab = (int)label, own = (int)self;
  f32x4 keep[KEEP ? KEEP : 1];
  // f(j, v, marked) over this thread's pieces v of columns j .. j + 3; with KEEP in registers, where f may replace them.  marked:
  // the label, a left-out column or padding is among the four; the others, nearly all, take no tests.
  auto visit = [&](auto f) {
    auto one = [&](int j, f32x4& v) {
      if ((uint32_t)(lab - j) < 4u || (uint32_t)(own - j) < 4u || j + 4 > B) f(j, v, std::true_type{});
      else f(j, v, std::false_type{});
    };
    if constexpr (KEEP > 0) {
#pragma unroll
      for (int u = 0; u < KEEP; ++u) {
        const int64_t q = threadIdx.x + u * SM_THREADS;
        if (q < nvec) one((int)q * 4, keep[u]);
      }
    } else {
      for (int64_t q = threadIdx.x; q < nvec; q += SM_THREADS) {
        f32x4 v = *reinterpret_cast<const f32x4*>(S + q * 4);
        one((int)q * 4, v);
      }
    }
  };
  auto counts = [&](int j, auto marked) { return !decltype(marked)::value || (j < B && j != own && j != lab); };
  if constexpr (KEEP > 0) {
#pragma unroll
    for (int u = 0; u < KEEP; ++u) {
      const int64_t q = threadIdx.x + u * SM_THREADS;
      if (q < nvec) keep[u] = *reinterpret_cast<const f32x4*>(S + q * 4);
    }
  }
  // the largest s v is s times the largest v, or with s < 0 the smallest
  const float up = s < 0.f ? -1.f : 1.f;
  float top = up * xl;
  visit([&](int j, f32x4& v, auto marked) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (counts(j + e, marked)) top = fmaxf(top, up * v[e]);
  });
  top = wave_reduce(top, [](float p, float q) { return fmaxf(p, q); });
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) red[0][wave] = top;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SM_WAVES; ++w) top = fmaxf(top, red[0][w]);
  const float mx = s * (up * top);
  float off = 0.f, ds = 0.f;
  visit([&](int j, f32x4& v, auto marked) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = 0.f;
      if (counts(j + e, marked)) {
        x = expf(fmaf(s, v[e], -mx));
        off += x;
        ds = fmaf(x, v[e] - xl, ds);
      }
      if constexpr (KEEP > 0) v[e] = x;
    }
  });
  auto plus = [](float p, float q) { return p + q; };
  off = wave_reduce(off, plus);
  ds = wave_reduce(ds, plus);
  if (lane == 0) { red[1][wave] = off; red[2][wave] = ds; }
  __syncthreads();
  off = red[1][0]; ds = red[2][0];
#pragma unroll
  for (int w = 1; w < SM_WAVES; ++w) { off += red[1][w]; ds += red[2][w]; }
  const float zl = s * xl, el = expf(fmaf(s, xl, -mx)), tot = off + el, inv = 1.f / tot;
  const float top_g = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(off * inv)));   // (the same in all lanes: scalar from here on)
  const int shift = half ? row_shift(top_g) : 0;
  const float m = half ? inv * (G_SCALE * power_of_two(shift)) : inv;
  visit([&](int j, f32x4& v, auto marked) {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = KEEP ? v[e] : counts(j + e, marked) ? expf(fmaf(s, v[e], -mx)) : 0.f;
      if (decltype(marked)::value && j + e == lab) x[e] = -off;
    }
    if (half) {
      store_unit_halves(G + j, a.gplane, x, m);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] *= m;
      store_unit_planes(G + j, a.gplane, x);
    }
  });
  if (threadIdx.x == 0) {
    // ce = log(tot) - (zl - mx); where the label holds most of the mass log1p(off / el) keeps the relative accuracy
    p.ce[a.r0 + i] = (el > 0.5f * tot) ? log1pf(off / el) : logf(tot) - (zl - mx);
    p.ds[a.r0 + i] = ds * inv;
    if (a.head) p.shift[i] = top_g == 0.f ? NO_ROW : (uint8_t)shift;
    if (shift) a.head->shifted = 1u;                                 // (whoever does stores the same)
  }
}

// The least exponent of the rows (0 if all are zeros) and whether there is another, the same in all threads; through LDS.
template <int NTHREADS>
__device__ __forceinline__ bool rows_differ(const uint8_t* shift, int64_t rows, char* smem, int& least) {
  int lo = NO_ROW, hi = -1;
  for (int64_t i = threadIdx.x * 4; i < rows; i += NTHREADS * 4) {   // (the array is whole pieces)
    const uint32_t v = *reinterpret_cast<const uint32_t*>(shift + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int x = (int)(v >> (8 * e) & 255u);
      if (i + e < rows && x != NO_ROW) { lo = min(lo, x); hi = max(hi, x); }
    }
  }
  lo = wave_reduce(lo, [](int x, int y) { return min(x, y); });
  hi = wave_reduce(hi, [](int x, int y) { return max(x, y); });
  int* red = reinterpret_cast<int*>(smem);
  if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = lo; red[16 + (threadIdx.x >> 6)] = hi; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NTHREADS / 64; ++w) { lo = min(lo, red[w]); hi = max(hi, red[16 + w]); }
  __syncthreads();
  least = __builtin_amdgcn_readfirstlane(hi < 0 ? 0 : lo);
  return lo < hi;
}

enum { SPLIT_KEY_WRITE = 0, SPLIT_KEY_ADD = 1, SPLIT_KEY_PARTS = 2 };

// Both gradient contractions, one T x T tile of one split per workgroup; query side first (workgroups < q_wgs, a multiple of
// 8), as in k_grads of mfma_kernels.hip.  NP: planes of a feature.
template <int T, int NP, int KMODE>
__global__ __launch_bounds__(Cfg<T>::NTHREADS) void k_split_grads(SplitArgs a, float cs) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  Acc<Cfg<T>::NFA> acc;
  // (all of it at once: a load for each of what follows costs a call of B = 8192, N = 8, d = 512 1.8 us of 202)
  const HalfHead head = a.head ? *a.head : HalfHead{};
  const bool half = head.half;
  // the sums of matrix m's features in their own units (the rows' powers of two on the query side: k_split_finalize)
  auto unscale = [&](int m) { return half ? (m ? head.unscale[1] : head.unscale[0]) * (1.f / G_SCALE) : 1.0f; };
  if ((int)blockIdx.x < a.q_wgs) {
    const int tiles = a.nMq * a.nN, total = tiles * a.nb * a.splitk;
    int lin;
    if (!xcd_linear(blockIdx.x, total, lin)) return;
    const int slice = lin / tiles, tile = lin % tiles;               // the workgroups of one slice read the same rows of Y
    const SplitBlock& p = a.z[slice / a.splitk];
    const int ks = slice % a.splitk;
    const int64_t i0 = (int64_t)(tile / a.nN) * T, k0 = (int64_t)(tile % a.nN) * T;
    const int kt0 = ks * a.ktps, left = (int)(a.Bp / BK) - kt0, kts = left < a.ktps ? left : a.ktps;
    const int ncols = a.dp - k0 < T ? (int)(a.dp - k0) : T;
    auto products = [&](auto ps) {
      using PS = decltype(ps);
      mainloop<T, FMT_K, FMT_R, false, true, PS>(p.G + i0 * a.Bp + (int64_t)kt0 * BK, a.Bp, p.Y + (int64_t)kt0 * BK * a.dp + k0, a.dp, kts * PS::N,
                                                 smem, acc, ncols, a.gplane, a.fplane);
    };
    if (half) products(HalfGrads<(NP + 1) / 2>{});
    else products(Planes<3, NP>{});
    store_tile_f32<T, false>(acc, smem, p.part + (int64_t)ks * a.bp * a.dp + i0 * a.dp + k0, a.dp, unscale(a.nb == 1 ? 0 : 1 - slice / a.splitk), ncols);
    return;
  }
  const int tiles = a.nMk * a.nN * a.key_splits, per_block = (tiles + 7) / 8 * 8;
  const int w = blockIdx.x - a.q_wgs, z = w / per_block;
  int lin;
  if (!xcd_linear(w - z * per_block, tiles, lin)) return;
  const SplitBlock& p = a.z[z];
  const int t2 = lin / a.nN, ks = t2 / a.nMk;
  const int64_t j0 = (int64_t)(t2 % a.nMk) * T, k0 = (int64_t)(lin % a.nN) * T;
  const int kt0 = ks * a.key_ktps, left = (int)(a.bp / BK) - kt0, kts = left < a.key_ktps ? left : a.key_ktps;
  const int ncols = a.dp - k0 < T ? (int)(a.dp - k0) : T;
  auto products = [&](auto ps, auto shifts) {
    using PS = decltype(ps);
    mainloop<T, FMT_R, FMT_R, false, true, PS, Whole, decltype(shifts)>(p.G + (int64_t)kt0 * BK * a.Bp + j0, a.Bp, p.X + (int64_t)kt0 * BK * a.dp + k0, a.dp,
                                                                        kts * PS::N, smem, acc, ncols, a.gplane, a.fplane, Whole{}, shifts);
  };
  // Rows of G with powers of two of their own: what they have in common is undone behind the sum, what they differ by goes into the features.
  // (Of fixed planes, the gradients of a batch whose positives have cosine 0.89 were off by 8e-4 at s = 40, 0.1 at 50 and were all zero from 70 on; now 5e-6
  // throughout.  us a call, bf16 planes / these with rows that differ / that do not: fp32 B = 8192, N = 8, d = 512 279 / 218 / 200; 4096, 16, 512
  // 81 / 77 / 70; 2048, 4, 512 77 / 77 / 63; 12288, 4, 256 762 / 567 / 534; bf16 12288, 8, 100 216 / 190 / 176.)
  if (half && head.shifted) {
    int least;
    if (rows_differ<Cfg<T>::NTHREADS>(p.shift, a.b, smem, least)) products(HalfGrads<(NP + 1) / 2>{}, RowShifts{p.shift + (int64_t)kt0 * BK, least});
    else products(HalfGrads<(NP + 1) / 2>{}, Unshifted{});
    const float common = power_of_two(-least);
#pragma unroll
    for (int i = 0; i < Cfg<T>::NFA; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] *= common;               // (on its own: with `unscale` below it can leave fp32's range)
  } else if (half) {
    products(HalfGrads<(NP + 1) / 2>{}, Unshifted{});
  } else {
    products(Planes<3, NP>{}, Unshifted{});
  }
  if constexpr (KMODE == SPLIT_KEY_PARTS) {
    store_tile_f32<T, false>(acc, smem, p.kpart + ((int64_t)ks * a.Bp + j0) * a.dp + k0, a.dp, unscale(z), ncols);
  } else {                                                           // (d % 4 == 0: a tile's last column piece is whole)
    const int cols = a.d - k0 < T ? (int)(a.d - k0) : T;
    const int64_t rows = a.B - j0;
    store_tile_f32<T, KMODE == SPLIT_KEY_ADD>(acc, smem, p.gk + j0 * a.d + k0, a.d, cs * unscale(z), cols, rows < T ? (int)rows : T);
  }
}

// Partial sums into the gradients: gX[row] += cs sum_ks part[ks][row] for the chunk's rows, and with PARTS also
// gY[j] = [add] gY[j] + cs sum_ks kpart[ks][j] for all rows; one wave per (matrix, row).  Workgroup 0 of the call's last chunk
// (scalars = 1) adds up loss and d/ds over the rank's rows instead, in fixed order.
// VEC: rows of the gradients can be written in 16-byte pieces.
template <bool PARTS, bool VEC>
__global__ __launch_bounds__(256) void k_split_finalize(SplitArgs a, float cs, float c, int add, int scalars, int accumulate, int64_t b_all,
                                                        float* loss, float* gs) {
  if (scalars && blockIdx.x == 0) {
    __shared__ float red[2][4];
    float l = 0.f, g = 0.f;
    for (int z = 0; z < a.nb; ++z)
      for (int64_t i0 = threadIdx.x; i0 < b_all; i0 += 1024) {
        float u[4], v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t i = i0 + q * 256;
          u[q] = i < b_all ? a.z[z].ce[i] : 0.f;
          v[q] = i < b_all ? a.z[z].ds[i] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) { l += u[q]; g += v[q]; }
      }
    for (int o = 32; o > 0; o >>= 1) { l += __shfl_xor(l, o); g += __shfl_xor(g, o); }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = l; red[1][threadIdx.x >> 6] = g; }
    __syncthreads();
    if (threadIdx.x == 0) {
      *loss = (accumulate ? *loss : 0.f) + c * ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]));
      *gs = (accumulate ? *gs : 0.f) + c * ((red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
    }
    return;
  }
  const int64_t rows = PARTS ? a.B : a.b;
  const int64_t w = ((int64_t)blockIdx.x - scalars) * 4 + (threadIdx.x >> 6);
  const int z = w >= rows ? 1 : 0;                                    // this wave's destination is block z's query side
  const int64_t row = w - z * rows;
  if (row >= rows || z >= a.nb) return;
  const SplitBlock& p = a.z[z];
  const SplitBlock& o = a.z[a.nb == 1 ? 0 : 1 - z];                   // whose key side lands in the same matrix
  const int64_t i = PARTS ? row - a.g0 : row, g = PARTS ? row : a.g0 + row;
  const bool own = i >= 0 && i < a.b;
  const uint8_t shift = own && a.head ? p.shift[i] : 0;               // (0 on bf16 planes)
  const float unscale = shift == NO_ROW ? 0.f : power_of_two(-(int)shift);
  float* out = p.gq + g * a.d;
  for (int64_t k = (threadIdx.x & 63) * 4; k < a.d; k += 256) {
    f32x4 u = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
    if (own)
      for (int ks = 0; ks < a.splitk; ++ks) u += *reinterpret_cast<const f32x4*>(p.part + ((int64_t)ks * a.bp + i) * a.dp + k);
    if constexpr (PARTS)
      for (int ks = 0; ks < a.key_splits; ++ks) v += *reinterpret_cast<const f32x4*>(o.kpart + ((int64_t)ks * a.Bp + row) * a.dp + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) u[e] = fmaf(u[e], unscale, v[e]);
    if constexpr (VEC) {
      f32x4 r = {0.f, 0.f, 0.f, 0.f};
      if (!PARTS || add) r = *reinterpret_cast<const f32x4*>(out + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = fmaf(cs, u[e], r[e]);
      *reinterpret_cast<f32x4*>(out + k) = r;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < a.d) out[k + e] = fmaf(cs, u[e], !PARTS || add ? out[k + e] : 0.f);
    }
  }
}

struct SplitPlan {
  int T;
  int64_t chunk;         // rows taken at a time
  int64_t bp, Bp, dp, frows;
  int nMq, nMk, nN, splitk, ktps, key_splits, key_ktps;
  bool parts;            // the key side goes through partial sums
  bool half;             // fp16 planes where the features allow them
  size_t off_head, off_planes, off_S, off_G, off_part, off_kpart, off_rows, off_shift, total;
  double us, exact_us;   // exact_us: of the best plan on bf16 planes
  int feature_planes(int np) const { return half && np == 1 ? 2 : np; }
};

// fp32 features in two fp16 planes lose the last bit of one value in four: about 2^-24 sqrt(2 / d) of a logit of unit rows, times s of an exponent.
// The lines lie where the gradients are as near to 64 bits as on bf16 planes (errors at B = 8192, N = 8, fp16 over bf16 planes, mean of 24 inputs, cosine 0.27: past
// the second d = 256, s = 60 / 80 / 100 0.99 / 1.04 / 1.07, 320, 100 1.05, 384, 90 1.05, 448, 100 1.04, and 192, 50 at 0.38 1.02; within it 512, 100 1.005;
// further ones at the top of this file); under the first the fp16 form gains little (us a call, bf16 / fp16 planes: B = 4096, N = 4, d = 64 73 / 70; 8192, 8, 128 136 / 127); calls past the second run six products on
// tiles and splits chosen for three (8192, 8, 320 184 at s = 1/0.07, 271 at 100; 12288, 4, 256 549 at 50, 831 at 100, planned for six 762).
bool halves_planned(int64_t d, int np) { return np == 1 || d >= 192; }
bool halves_hold(float s, int64_t d, int np) { return np == 1 || 5.f * fabsf(s) <= (float)d; }

int64_t round_up(int64_t v, int64_t u) { return (v + u - 1) / u * u; }

void split_layout(SplitPlan& pl, int64_t b, int nb, int np) {
  size_t o = 0;
  pl.off_head = o;
  if (pl.half) o += HEAD_BYTES;
  pl.off_planes = o; o += 2 * align_up((size_t)pl.feature_planes(np) * pl.frows * pl.dp * 2);
  pl.off_S = o;      o += nb * align_up((size_t)pl.bp * pl.Bp * 4);
  pl.off_G = o;      o += nb * align_up((size_t)3 * pl.bp * pl.Bp * 2);
  pl.off_part = o;   o += nb * align_up((size_t)pl.splitk * pl.bp * pl.dp * 4);
  pl.off_kpart = o;
  if (pl.parts) o += nb * align_up((size_t)pl.key_splits * pl.Bp * pl.dp * 4);
  pl.off_rows = o;   o += 2 * nb * align_up((size_t)b * 4);
  pl.off_shift = o;
  if (pl.half) o += nb * align_up((size_t)pl.bp);
  pl.total = o;
}

// Compares estimated times over tile sizes and splits, for one chunk of rows.  (Rows of the gradients that are not whole
// 16-byte pieces go through partial sums: the tile store writes such pieces.)
SplitPlan make_split_plan(int64_t B, int64_t d, int64_t b, int nb, int np, int64_t chunk, bool half) {
  static const int Q_SPLITS[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}, K_SPLITS[] = {1, 2, 3, 4, 6, 8};
  SplitPlan best;
  best.us = 1e300;
  // the tile loop's quotient of a step by the pieces of a reduction taken in sweeps (mfma_tile.h) is exact below 2^32 steps times pieces
  // (it first fails at 37927 pieces and three sweeps); logits have 1024 pieces at most
  constexpr int64_t SWEEP_PIECES_MOST = 32768;
  static_assert(HalfGrads<2>::N * SWEEP_PIECES_MOST * SWEEP_PIECES_MOST < (int64_t)1 << 32);
  const int nl = np == 1 ? 1 : half ? 4 : 6, ng = np == 3 ? (half ? 3 : 6) : half ? 2 : 3;
  for (int T = 128; T <= 256; T += 128) {
    SplitPlan pl;
    pl.T = T; pl.chunk = chunk; pl.half = half;
    pl.bp = round_up(chunk, T); pl.Bp = round_up(B, T); pl.dp = round_up(d, BK);
    pl.frows = pl.Bp + (chunk < b ? pl.bp : T);                      // a rank's last tile (chunk) may reach past the last row
    pl.nMq = (int)(pl.bp / T); pl.nMk = (int)(pl.Bp / T); pl.nN = (int)((pl.dp + T - 1) / T);
    const double slots = T == 256 ? CHIP_CUS : 2 * CHIP_CUS, fix = T == 256 ? 8.0 : 3.0;
    const double lt = (double)nb * pl.nMq * pl.nMk, lrounds = (double)(int64_t)((lt + slots - 1) / slots);
    const double logits = lrounds * ((double)(pl.dp / BK) * nl * step_us(T, lt) + fix);
    const double bytes = (double)nb * pl.bp * pl.Bp;
    const double base = logits + (half ? 16.0 : 20.0) * bytes / BYTES_PER_US + (pl.feature_planes(np) * 2 + 4) * 2.0 * pl.frows * pl.dp / BYTES_PER_US;
    const int kq = (int)(pl.Bp / BK), kk = (int)(pl.bp / BK);
    for (int sk : Q_SPLITS) {
      if (sk > kq) break;
      pl.ktps = (kq + sk - 1) / sk; pl.splitk = (kq + pl.ktps - 1) / pl.ktps;
      if (half && pl.ktps > SWEEP_PIECES_MOST) continue;
      for (int ks : K_SPLITS) {
        if (ks > kk) break;
        pl.key_ktps = (kk + ks - 1) / ks; pl.key_splits = (kk + pl.key_ktps - 1) / pl.key_ktps;
        if (half && pl.key_ktps > SWEEP_PIECES_MOST) continue;
        pl.parts = pl.key_splits > 1 || d % 4 != 0;
        const double nq = (double)nb * pl.nMq * pl.nN * pl.splitk, nk = (double)nb * pl.nMk * pl.nN * pl.key_splits;
        const double step = step_us(T, nq + nk), lq = pl.ktps * ng * step + fix, lk = pl.key_ktps * ng * step + fix;
        const double longest = lq > lk ? lq : lk;
        const double grads = nq + nk <= slots ? longest : (nq * lq + nk * lk) / slots + 0.5 * longest;
        const double part = 8.0 * nb * pl.bp * pl.dp * pl.splitk, key = 4.0 * nb * pl.Bp * pl.dp;
        pl.us = base + grads + (part + (pl.parts ? 2.0 * key * pl.key_splits + key : key)) / BYTES_PER_US + 25.0;
        if (pl.us < best.us) { split_layout(pl, b, nb, np); best = pl; }
      }
    }
  }
  return best;
}

template <class K>
bool allow_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <int T>
constexpr int SPLIT_SMEM = OUT_SMEM_BYTES<T> > Cfg<T>::SMEM_BYTES ? OUT_SMEM_BYTES<T> : Cfg<T>::SMEM_BYTES;

template <int T, int NP>
bool raise_lds() {
  return allow_lds(k_split_logits<T, NP>, SPLIT_SMEM<T>) && allow_lds(k_split_grads<T, NP, SPLIT_KEY_WRITE>, SPLIT_SMEM<T>) &&
                         allow_lds(k_split_grads<T, NP, SPLIT_KEY_ADD>, SPLIT_SMEM<T>) && allow_lds(k_split_grads<T, NP, SPLIT_KEY_PARTS>, SPLIT_SMEM<T>);
}

template <int T, int NP>
void split_products(bool grads, bool parts, bool add, const SplitArgs& a, float cs, hipStream_t st) {
  if (!grads) {
    const int nI = (int)(a.bp / T), nJ = (int)(a.Bp / T);
    const int sbi = nI < 8 ? nI : 8, sbj = 32 / sbi < nJ ? 32 / sbi : nJ;
    k_split_logits<T, NP><<<dim3((unsigned)(a.nb * ((nI * nJ + 7) / 8 * 8))), Cfg<T>::NTHREADS, SPLIT_SMEM<T>, st>>>(a, sbi, sbj);
    return;
  }
  const dim3 grid((unsigned)(a.q_wgs + a.nb * ((a.nMk * a.nN * a.key_splits + 7) / 8 * 8)));
  auto go = [&](auto kernel) { kernel<<<grid, Cfg<T>::NTHREADS, SPLIT_SMEM<T>, st>>>(a, cs); };
  if (parts) go(k_split_grads<T, NP, SPLIT_KEY_PARTS>);
  else if (add) go(k_split_grads<T, NP, SPLIT_KEY_ADD>);
  else go(k_split_grads<T, NP, SPLIT_KEY_WRITE>);
}

template <int DT>
int split_run_typed(const Problem& pr, const SplitPlan& pl) {
  constexpr int NP = DT == DISCO_BF16 ? 1 : 3;
  const int nb = loss_blocks(pr.variant);
  char* ws = static_cast<char*>(pr.ws);
  const float c = loss_norm(pr.B, pr.variant), cs = c * pr.s;
  hipStream_t st = pr.stream;
  auto aligned = [](const void* p, size_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
  const bool fvec = pr.d % 4 == 0 && aligned(pr.I, DT == DISCO_BF16 ? 8 : 16) && aligned(pr.T, DT == DISCO_BF16 ? 8 : 16);
  const bool gvec = pr.d % 4 == 0 && aligned(pr.gI, 16) && aligned(pr.gT, 16);
  uint16_t* planes[2];
  for (int z = 0; z < 2; ++z) planes[z] = reinterpret_cast<uint16_t*>(ws + pl.off_planes + z * align_up((size_t)pl.feature_planes(NP) * pl.frows * pl.dp * 2));
  HalfHead* head = nullptr;

  stage_mark(st, 0);
  {
    const int64_t pieces = nb * pl.frows * (pl.dp >> 2);
    dim3 grid((unsigned)(pieces < 4096 * 256 ? (pieces + 255) / 256 : 4096));
    uint32_t* flags = nullptr;
    int nflags = 0;
    // (the gradients' scale is a power of two down to 2^-95 times cs, which has to stay a normal number)
    if (pl.half && (cs == 0.f || fabsf(cs) >= 0x1p-30f) && halves_hold(pr.s, pr.d, NP)) {
      head = reinterpret_cast<HalfHead*>(ws + pl.off_head);
      flags = reinterpret_cast<uint32_t*>(ws + pl.off_head + align_up(sizeof(HalfHead)));
      const int lanes = pl.dp <= 128 ? 16 : 64;
      const int64_t groups = (nb * pl.frows * lanes + 255) / 256;
      nflags = (int)(groups < HALF_FLAGS ? groups : HALF_FLAGS);
      auto halves = [&](auto kernel) { kernel<<<dim3((unsigned)nflags), 256, 0, st>>>(pr.I, pr.T, pr.B, pr.d, pl.frows, pl.dp, nb, planes[0], planes[1], head, flags); };
      if (fvec) { if (lanes == 16) halves(k_feature_halves<DT, true, 16>); else halves(k_feature_halves<DT, true, 64>); }
      else { if (lanes == 16) halves(k_feature_halves<DT, false, 16>); else halves(k_feature_halves<DT, false, 64>); }
    }
    // Behind the halves these workgroups nearly always have nothing to do, and where they have, 1024 take no longer than 4096, which cost other calls
    // 1 us more.  (us a call whose features leave fp16's range, bf16 planes alone / 256 workgroups / 1024: fp32 B = 8192, N = 8, d = 512, norms
    // from 2^-10 to 1 301 / 327 / 321, one row 100 times longer 307 / 333 / 327, a first row of zeros 305 / 331 / 312; 4096, 16, 512 86 / 101 / 98, 86 / 103 / 99, 87 / 103 / 93.
    // What is left is the launch, the halves up to where it shows, and tiles and splits chosen for three products where six run.)
    if (head && grid.x > 1024) grid.x = 1024;
    auto exact = [&](auto kernel) { kernel<<<grid, 256, 0, st>>>(pr.I, pr.T, pr.B, pr.d, pl.frows, pl.dp, nb, planes[0], planes[1], head, flags, nflags); };
    if (fvec) exact(k_feature_planes<DT, true>);
    else exact(k_feature_planes<DT, false>);
  }
  for (int64_t r0 = 0; r0 < pr.b; r0 += pl.chunk) {
    const bool last = r0 + pl.chunk >= pr.b, add = pr.accumulate || r0 > 0;
    SplitArgs a;
    a.b = last ? pr.b - r0 : pl.chunk; a.bp = pl.bp; a.B = pr.B; a.Bp = pl.Bp; a.d = pr.d; a.dp = pl.dp;
    a.g0 = (int64_t)pr.rank * pr.b + r0; a.r0 = r0;
    a.fplane = pl.frows * pl.dp; a.gplane = pl.bp * pl.Bp;
    a.nb = nb; a.variant = pr.variant; a.head = head;
    a.nMq = pl.nMq; a.nMk = pl.nMk; a.nN = pl.nN;
    a.splitk = pl.splitk; a.ktps = pl.ktps; a.key_splits = pl.key_splits; a.key_ktps = pl.key_ktps;
    a.q_wgs = (nb * a.nMq * a.nN * a.splitk + 7) / 8 * 8;
    for (int z = 0; z < 2; ++z) {
      SplitBlock& p = a.z[z];
      p.X = planes[z] + a.g0 * pl.dp;
      p.Y = planes[nb == 1 ? z : 1 - z];
      const int zz = z < nb ? z : 0;
      p.S = reinterpret_cast<float*>(ws + pl.off_S + zz * align_up((size_t)pl.bp * pl.Bp * 4));
      p.G = reinterpret_cast<uint16_t*>(ws + pl.off_G + zz * align_up((size_t)3 * pl.bp * pl.Bp * 2));
      p.shift = pl.half ? reinterpret_cast<uint8_t*>(ws + pl.off_shift + zz * align_up((size_t)pl.bp)) : nullptr;
      p.part = reinterpret_cast<float*>(ws + pl.off_part + zz * align_up((size_t)pl.splitk * pl.bp * pl.dp * 4));
      p.kpart = pl.parts ? reinterpret_cast<float*>(ws + pl.off_kpart + zz * align_up((size_t)pl.key_splits * pl.Bp * pl.dp * 4)) : nullptr;
      p.ce = reinterpret_cast<float*>(ws + pl.off_rows + (2 * zz) * align_up((size_t)pr.b * 4));
      p.ds = reinterpret_cast<float*>(ws + pl.off_rows + (2 * zz + 1) * align_up((size_t)pr.b * 4));
      p.gq = z == 0 ? pr.gI : pr.gT;
      p.gk = z == 0 ? pr.gT : pr.gI;
    }
    if (pl.T == 256) split_products<256, NP>(false, pl.parts, add, a, cs, st);
    else split_products<128, NP>(false, pl.parts, add, a, cs, st);
    if (r0 == 0) stage_mark(st, 1);
    const dim3 rows((unsigned)pl.bp, (unsigned)nb);
    if (pl.Bp <= (int64_t)SM_THREADS * 4 * 4) k_split_softmax<4><<<rows, SM_THREADS, 0, st>>>(a, pr.s);
    else if (pl.Bp <= (int64_t)SM_THREADS * 8 * 4) k_split_softmax<8><<<rows, SM_THREADS, 0, st>>>(a, pr.s);
    else if (pl.Bp <= (int64_t)SM_THREADS * 16 * 4) k_split_softmax<16><<<rows, SM_THREADS, 0, st>>>(a, pr.s);
    else k_split_softmax<0><<<rows, SM_THREADS, 0, st>>>(a, pr.s);
    if (r0 == 0) { stage_mark(st, 2); stage_mark(st, 3); }
    if (pl.T == 256) split_products<256, NP>(true, pl.parts, add, a, cs, st);
    else split_products<128, NP>(true, pl.parts, add, a, cs, st);
    if (last) stage_mark(st, 4);
    const int64_t frows = nb * (pl.parts ? pr.B : a.b);
    const int sc = last ? 1 : 0;
    auto fin = [&](auto kernel) {
      kernel<<<dim3((unsigned)((frows + 3) / 4 + sc)), 256, 0, st>>>(a, cs, c, add ? 1 : 0, sc, pr.accumulate, pr.b, pr.loss, pr.gs);
    };
    if (pl.parts) { if (gvec) fin(k_split_finalize<true, true>); else fin(k_split_finalize<true, false>); }
    else fin(k_split_finalize<false, true>);
  }
  stage_mark(st, 5);
  return hipGetLastError() == hipSuccess ? DISCO_OK : DISCO_ERR_HIP;
}

// fp16 planes are one more launch and one more plane of the features than their products read as leading ones, and the estimates overrate
// short calls' products: by how much their plan has to be the shorter one.  (us a call, bf16 / fp16 planes, by the estimates' difference: fp32 features 7.6: 47.9 / 46.8;
// 11 51.0 / 48.0; 12 51.1 / 50.6; 14 57.1 / 52.2; bf16 features 6.0: 54.4 / 60.2; 10 59.3 / 60.5; 12 76.0 / 77.9; 14.5 58.5 / 60.4; 16.4 98.8 / 96.6; 19 84.0 / 79.6;
// 25 94.0 / 90.0.)
double half_allowance_us(int np) { return np == 3 ? 6.0 : 16.0; }

// The plan whose rows are taken in as few chunks as keep the workspace within `limit` (0 bytes in `total`: there is none).
SplitPlan compare_within(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit) {
  const int np = dtype == DISCO_BF16 ? 1 : 3;
  for (int64_t chunks = 1;; chunks *= 2) {
    const int64_t chunk = chunks == 1 ? b : round_up((b + chunks - 1) / chunks, 256);
    SplitPlan pl = make_split_plan(B, d, b, nb, np, chunk, false);
    pl.exact_us = pl.us;
    if (pl.total <= limit) {
      if (!halves_planned(d, np)) return pl;
      SplitPlan hp = make_split_plan(B, d, b, nb, np, chunk, true);
      hp.exact_us = pl.us;
      return hp.total <= limit && hp.us + half_allowance_us(np) < pl.us ? hp : pl;
    }
    if (chunk <= 256) { pl.total = 0; return pl; }
  }
}

SplitPlan plan_within(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit) {
  static thread_local PlanCache<SplitPlan, 6> cache;
  return cache.get({B, d, b, dtype, nb, (int64_t)limit}, [&] { return compare_within(B, d, b, dtype, nb, limit); });
}

}  // namespace

bool split_supported(int64_t B, int64_t b) { return B <= ((int64_t)1 << 22) && b >= 1; }   // 32-bit lane offsets over 256 rows of pitch B

bool split_aligned(const Problem& pr) {
  return pr.d % 4 != 0 || ((reinterpret_cast<uintptr_t>(pr.gI) | reinterpret_cast<uintptr_t>(pr.gT)) & 15u) == 0;
}

// (The model ranks plans; its sum of the parts is this much more than what a call takes: 402 against 313 us at B = 8192,
// N = 8, d = 512, 113 against 87 at 4096, 16, 512, 43 against 33 at 2048, 16, d = 200 in bf16.)
constexpr double MODEL_SHARE = 0.77;
static double chunks_of(const SplitPlan& pl, int64_t b) { return (double)((b + pl.chunk - 1) / pl.chunk); }

// What the choice against the small kernels goes by: the time on bf16 planes, which the line between them was measured with (and which a call
// takes whose features fp16 cannot hold).
double split_estimate_us(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit, size_t* bytes) {
  const SplitPlan pl = plan_within(B, d, b, dtype, nb, limit);
  *bytes = pl.total;
  return MODEL_SHARE * pl.exact_us * chunks_of(pl, b);
}

bool split_raise_lds() { return raise_lds<128, 1>() && raise_lds<128, 3>() && raise_lds<256, 1>() && raise_lds<256, 3>(); }

void split_describe(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit, disco_plan* out) {
  const SplitPlan pl = plan_within(B, d, b, dtype, nb, limit);
  out->kernels = DISCO_KERNELS_SPLIT;
  out->logit_tile = out->gradient_tile = pl.T;
  out->row_chunks = (int)((b + pl.chunk - 1) / pl.chunk);
  out->key_panels = 1;
  out->query_splits = pl.splitk;
  out->key_splits = pl.key_splits;
  out->microseconds = MODEL_SHARE * pl.us * chunks_of(pl, b);
}

int split_run(const Problem& pr, size_t limit) {
  const SplitPlan pl = plan_within(pr.B, pr.d, pr.b, pr.dtype, loss_blocks(pr.variant), limit);
  return pr.dtype == DISCO_BF16 ? split_run_typed<DISCO_BF16>(pr, pl) : split_run_typed<DISCO_F32>(pr, pl);
}

}  // namespace disco

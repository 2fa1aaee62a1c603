// The fp32 path: fp32 arithmetic on the matrix instructions, any shape, either input dtype (large calls: split_kernels.hip).
// The two b x B blocks of raw similarities live in the workspace in fp32 (the 2B^2/N memory model
// of Sec. 4.1) and are turned in place into (softmax - onehot); the four gradient contractions of
// Eq. 4-6 are plain tiled products.  Everything is deterministic (no float atomics).
#include "common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace disco {
namespace {

__device__ __forceinline__ float block_reduce(float v, bool is_max, float* red) {
  for (int o = 32; o > 0; o >>= 1) {
    float w = __shfl_xor(v, o);
    v = is_max ? fmaxf(v, w) : v + w;
  }
  int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float r = red[0];
  for (int w = 1; w < (int)(blockDim.x / 64); ++w) r = is_max ? fmaxf(r, red[w]) : r + red[w];
  return r;
}

// One pass of a workgroup over a row of B floats: x <- f(j, x) for every column j (stored back if WRITE).  The row
// starts at any float offset of a 256-byte aligned buffer: `head` (0..3) columns up to the first 16-byte boundary,
// then 16-byte pieces, then up to 3 columns; the at most six odd columns go one per thread.
template <bool WRITE, class F>
__device__ __forceinline__ void row_visit(float* w, int64_t B, int head, F f) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const int64_t nvec = (B - head) >> 2;
  for (int64_t q = threadIdx.x; q < nvec; q += 256) {
    f32x4* p = reinterpret_cast<f32x4*>(w + head) + q;
    f32x4 v = *p;
    const int64_t j = head + q * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = f(j + e, v[e]);
    if (WRITE) *p = v;
  }
  const int64_t t0 = head + nvec * 4;
  const int nrest = head + (int)(B - t0);
  if ((int)threadIdx.x < nrest) {
    const int64_t j = (int)threadIdx.x < head ? (int64_t)threadIdx.x : t0 + ((int)threadIdx.x - head);
    const float x = f(j, w[j]);
    if (WRITE) w[j] = x;
  }
}

// Step 2 (Alg. 1 cross_entropy_loss, and the softmax gradient of loss.backward()).  One workgroup per
// local row: lse_i = m + log(sum exp(z - m)) over z = s * W[i][:], ce_i = lse_i - z[label], then
// W[i][j] <- P_ij - [j = label].  The off-label mass is summed on its own so that P_label - 1 is
// formed as -(sum of the other terms)/(total) without cancellation.  Also the row's share of
// d/ds:  sum_j (P_ij - [j=label]) * W_ij.
// variant LOSS_NTXENT: the positive is the other view's row and column `self` (the row itself) takes no part:
// it is left out of the maximum and the sums and its gradient entry is 0.
__global__ __launch_bounds__(256) void naive_row_softmax(float* ws, int64_t b, int64_t B, int64_t pitch, int rank, float s,
                                                          float* row_ce, float* row_ds, int variant) {
  __shared__ float red[4];
  const int z = blockIdx.y;
  const int64_t i = blockIdx.x;
  const int64_t row0 = ((int64_t)z * b + i) * pitch;
  float* w = ws + row0;
  const int64_t to_boundary = (4 - (row0 & 3)) & 3;
  const int head = (int)(to_boundary < B ? to_boundary : B);
  const int64_t label = label_row((int64_t)rank * b + i, B, variant);
  const int64_t self = masked_col((int64_t)rank * b + i, variant);
  float mx = -INFINITY;
  row_visit<false>(w, B, head, [&](int64_t j, float x) {
    if (j != self) mx = fmaxf(mx, s * x);
    return x;
  });
  mx = block_reduce(mx, true, red);
  float off = 0.f;
  row_visit<false>(w, B, head, [&](int64_t j, float x) {
    if (j != label && j != self) off += expf(s * x - mx);
    return x;
  });
  off = block_reduce(off, false, red);
  const float zl = s * w[label];
  const float el = expf(zl - mx);
  const float tot = off + el;
  const float inv = 1.f / tot;
  float ds = 0.f;
  row_visit<true>(w, B, head, [&](int64_t j, float x) {
    const float g = (j == label) ? -off * inv : (j == self) ? 0.f : expf(s * x - mx) * inv;
    ds = fmaf(g, x, ds);
    return g;
  });
  ds = block_reduce(ds, false, red);
  if (threadIdx.x == 0) {
    // ce = log(tot) - (zl - mx).  When the label holds most of the mass this is log1p(off/el), which
    // keeps relative accuracy for a saturated softmax (s = 100) where the plain difference cancels.
    row_ce[(size_t)z * b + i] = (el > 0.5f * tot) ? log1pf(off / el) : logf(tot) - (zl - mx);
    row_ds[(size_t)z * b + i] = ds;
  }
}

// The same for rows of up to 2048 columns that start on a 16-byte boundary: one wave per row, which it keeps in registers (V pieces
// of four columns per lane), so that the row is read and written once and no barrier stands between its sums.  What bounds such a
// launch is that chain of sums.  (us a call, workgroups per row / waves: fp32 B = 256, N = 4, d = 512: 17.6 / 16.2; 600 pairs of views, N = 3, d = 77:
// 19.8 / 18.4; bf16 B = 1024, N = 2, d = 256: 37.6 / 36.6; 256 two-view rows: 19.2 / 17.0.)
constexpr int WAVE_ROW_COLUMNS = 2048;

template <int V>
__global__ __launch_bounds__(256) void naive_wave_softmax(float* ws, int64_t b, int64_t B, int64_t pitch, int nb, int rank, float s,
                                                          float* row_ce, float* row_ds, int variant) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= nb * b) return;
  const int64_t g = (int64_t)rank * b + (row >= b ? row - b : row);
  const int label = (int)label_row(g, B, variant), self = (int)masked_col(g, variant), n = (int)B;
  float* w = ws + row * pitch;
  const float xl = w[label];
  f32x4 x[V], e[V];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int j = (lane + 64 * u) * 4;
    if (j < n) x[u] = *reinterpret_cast<const f32x4*>(w + j);          // (up to three columns of the pitch behind the row)
  }
#pragma unroll
  for (int u = 0; u < V; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = (lane + 64 * u) * 4 + k;
      if (j < n && j != self) mx = fmaxf(mx, s * x[u][k]);
    }
  mx = wave_reduce(mx, [](float a, float c) { return fmaxf(a, c); });
  auto sum = [](float a, float c) { return a + c; };
  float off = 0.f;
#pragma unroll
  for (int u = 0; u < V; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = (lane + 64 * u) * 4 + k;
      e[u][k] = expf(s * x[u][k] - mx);
      if (j < n && j != label && j != self) off += e[u][k];
    }
  off = wave_reduce(off, sum);
  const float zl = s * xl, el = expf(zl - mx), tot = off + el, inv = 1.f / tot;
  float ds = 0.f;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    f32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = (lane + 64 * u) * 4 + k;
      v[k] = j == label ? -off * inv : j == self ? 0.f : e[u][k] * inv;
      if (j < n) ds = fmaf(v[k], x[u][k], ds);
    }
    const int j = (lane + 64 * u) * 4;
    if (j < n) *reinterpret_cast<f32x4*>(w + j) = v;
  }
  ds = wave_reduce(ds, sum);
  if (lane == 0) {
    row_ce[row] = (el > 0.5f * tot) ? log1pf(off / el) : logf(tot) - (zl - mx);
    row_ds[row] = ds;
  }
}

// ------------------------------------------------------------------------------------------------
// Small calls: the same four contractions in two launches around the softmax, on 32 R x 32 R output tiles (R = 1 or 2).
// What bounds such a call is latency: launches, and the reduction that one workgroup walks alone (a rank of B = 256,
// N = 4, d = 512 is four 128 x 128 similarity tiles, each a chain of 32 LDS round trips).  So the tiles are small, the
// NW waves of a workgroup split the reduction among them and load their operands from memory straight into the
// registers of the fp32 matrix instruction (no LDS, no barrier until the partial tiles are added up at the end), and
// the next piece's loads are in flight while one is multiplied.  Key side and query side share a launch: a tile of
// gradient rows adds up both (the query side only where the rows are the rank's own), so every row has one writer.

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Four consecutive values from element idx on.  VEC: they start on a 16-byte boundary.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* base, int64_t idx) {
  if constexpr (VEC) return *reinterpret_cast<const f32x4*>(base + idx);
  return f32x4{base[idx], base[idx + 1], base[idx + 2], base[idx + 3]};
}

__device__ __forceinline__ int upper_half() { return (threadIdx.x >> 5) & 1; }

// acc[u][v] += sum over k in [k0, k1) of A(row block u, k) B(k, column block v), one value of each operand per lane and
// instruction: the lanes of the lower half supply reduction indices k .. k + 3 of an 8-deep piece, the upper half
// k + 4 .. k + 7 (any assignment does as long as both operands share it).  A.get4(u, k) / B.get4(v, k): this lane's four
// values of row (column) block u of the piece that starts at k, the same k in all lanes; get1(u, k): the value at k.
template <int R, class LA, class LB>
__device__ __forceinline__ void wave_product(f32x16 (&acc)[R][R], int64_t k0, int64_t k1, const LA& A, const LB& B) {
  constexpr int U = 4;                                  // 8-deep pieces fetched at a time
  struct Regs { f32x4 a[U][R], b[U][R]; };
  auto fetch = [&](Regs& g, int64_t k) {
#pragma unroll
    for (int c = 0; c < U; ++c)
#pragma unroll
      for (int u = 0; u < R; ++u) { g.a[c][u] = A.get4(u, k + c * 8); g.b[c][u] = B.get4(u, k + c * 8); }
  };
  int64_t k = k0;
  if (k + 8 * U <= k1) {
    Regs cur;
    fetch(cur, k);
    for (;;) {
      const bool more = k + 16 * U <= k1;
      Regs nxt;
      if (more) fetch(nxt, k + 8 * U);
#pragma unroll
      for (int c = 0; c < U; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int u = 0; u < R; ++u)
#pragma unroll
            for (int v = 0; v < R; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(cur.a[c][u][e], cur.b[c][v][e], acc[u][v], 0, 0, 0);
      k += 8 * U;
      if (!more) break;
      cur = nxt;
    }
  }
  for (; k < k1; k += 8) {                              // what is left, element by element: past k1 both operands count as 0
    float a[R][4], b[R][4];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t kk = k + upper_half() * 4 + e, kc = kk < k1 ? kk : k1 - 1;
        const float x = A.get1(u, kc), y = B.get1(u, kc);
        a[u][e] = kk < k1 ? x : 0.f;
        b[u][e] = kk < k1 ? y : 0.f;
      }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < R; ++u)
#pragma unroll
        for (int v = 0; v < R; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][e], b[v][e], acc[u][v], 0, 0, 0);
  }
}

// Adds up the waves' partial tiles in wave order and hands every entry to out(row, column, value), rows and columns
// relative to the tile; 32 consecutive columns per half-wave.
template <int R, int NW, class FOut>
__device__ __forceinline__ void join_waves(const f32x16 (&acc)[R][R], float (*red)[R * R * 16][64], FOut out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < R; ++u)
#pragma unroll
    for (int v = 0; v < R; ++v)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[wave][(u * R + v) * 16 + r][lane] = acc[u][v][r];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < R * R * 16 / NW; ++q) {
    const int idx = q * NW + wave, uv = idx >> 4, r = idx & 15;
    float s = red[0][idx][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w][idx][lane];
    out((uv / R) * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), (uv % R) * 32 + (lane & 31), s);
  }
}

template <int R, int C>
__device__ __forceinline__ void clear(f32x16 (&acc)[R][C]) {
#pragma unroll
  for (int u = 0; u < R; ++u)
#pragma unroll
    for (int v = 0; v < C; ++v)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[u][v][r] = 0.f;
}

// This wave's part [k0, k1) of a reduction of length K (8-deep pieces dealt in runs).
template <int NW>
__device__ __forceinline__ void wave_range(int64_t K, int64_t& k0, int64_t& k1) {
  const int64_t per = ((K + 7) / 8 + NW - 1) / NW * 8;
  k0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * per;
  k1 = k0 + per < K ? k0 + per : K;
}

// Operand whose reduction index is contiguous: element (row, k) at base[row ld + k], one row per lane and block.
template <bool VEC, int R>
struct AlongK {
  const float* base;
  int64_t off[R];
  __device__ __forceinline__ AlongK(const float* p, int64_t ld, int64_t row0, int64_t rows) : base(p) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int64_t row = row0 + u * 32 + (threadIdx.x & 31);
      off[u] = (row < rows ? row : rows - 1) * ld;       // a row past the end repeats the last; its results are not stored
    }
  }
  __device__ __forceinline__ f32x4 get4(int u, int64_t k) const { return load4<VEC>(base, off[u] + upper_half() * 4 + k); }
  __device__ __forceinline__ float get1(int u, int64_t k) const { return base[off[u] + k]; }
};
// Operand whose row (column) index is contiguous: element (k, col) at base[k ld + col].
template <int R>
struct AcrossK {
  const float* base;
  int64_t ld, col[R], up;
  __device__ __forceinline__ AcrossK(const float* p, int64_t pitch, int64_t col0, int64_t cols) : base(p), ld(pitch), up(upper_half() * 4 * pitch) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int64_t c = col0 + u * 32 + (threadIdx.x & 31);
      col[u] = c < cols ? c : cols - 1;
    }
  }
  __device__ __forceinline__ float get1(int u, int64_t k) const { return base[k * ld + col[u]]; }
  __device__ __forceinline__ f32x4 get4(int u, int64_t k) const {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = base[(k + e) * ld + (col[u] + up)];
    return v;
  }
};
// Rows of the gradient matrix of the rank's own rows, by global row: rows of other ranks that share the tile count as 0.
// VEC: the pitch is a multiple of 4 floats.
template <bool VEC, int R>
struct OwnRows {
  AlongK<VEC, R> rows;
  bool own[R];
  __device__ __forceinline__ OwnRows(const float* W, int64_t pitch, int64_t local0, int64_t b)
      : rows(W, pitch, 0, 1) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int64_t i = local0 + u * 32 + (threadIdx.x & 31);
      own[u] = i >= 0 && i < b;
      rows.off[u] = (own[u] ? i : 0) * pitch;
    }
  }
  __device__ __forceinline__ f32x4 get4(int u, int64_t k) const {
    const f32x4 v = rows.get4(u, k);
    return own[u] ? v : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ float get1(int u, int64_t k) const { const float v = rows.get1(u, k); return own[u] ? v : 0.f; }
};

struct SmallShape {
  int64_t b, B, d, pitch;        // pitch: floats between the rows of a block's matrix
  int rank, nb, variant, accumulate;
  int out_pairs;                 // rows of the gradients can be written in 8-byte pieces
};
// loss and d/ds from the rows' shares, by one workgroup in fixed order.  red: 2 NW floats of LDS.
template <int NW>
__device__ __forceinline__ void small_scalars(const SmallShape& f, float c, const float* row_ce, const float* row_ds, float* loss, float* gs,
                                              float* red) {
  float a = 0.f, g = 0.f;
  for (int64_t i = threadIdx.x; i < f.nb * f.b; i += 64 * NW) { a += row_ce[i]; g += row_ds[i]; }
  for (int o = 32; o > 0; o >>= 1) { a += __shfl_xor(a, o); g += __shfl_xor(g, o); }
  if ((threadIdx.x & 63) == 0) { red[2 * (threadIdx.x >> 6)] = a; red[2 * (threadIdx.x >> 6) + 1] = g; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) { a += red[2 * w]; g += red[2 * w + 1]; }
    *loss = (f.accumulate ? *loss : 0.f) + c * a;
    *gs = (f.accumulate ? *gs : 0.f) + c * g;
  }
}

template <bool VEC, int R, int NW>
__global__ __launch_bounds__(64 * NW) void small_similarity(const float* I, const float* T, SmallShape f, float* ws) {
  __shared__ float red[NW][R * R * 16][64];
  const int z = blockIdx.z;
  const int64_t m0 = (int64_t)blockIdx.y * 32 * R, n0 = (int64_t)blockIdx.x * 32 * R;
  const AlongK<VEC, R> A((z == 0 ? I : T) + f.rank * f.b * f.d, f.d, m0, f.b), Bm(z == 0 ? T : I, f.d, n0, f.B);
  f32x16 acc[R][R];
  clear(acc);
  int64_t k0, k1;
  wave_range<NW>(f.d, k0, k1);
  wave_product<R>(acc, k0, k1, A, Bm);
  float* W = ws + (size_t)z * f.b * f.pitch;
  join_waves<R, NW>(acc, red, [&](int r, int c, float v) {
    if (m0 + r < f.b && n0 + c < f.B) W[(m0 + r) * f.pitch + n0 + c] = v;
  });
}

// The same on 16 x 16 tiles (16 x 16 x 4 products: four groups of 16 lanes supply 4 reduction indices each of a 16-deep piece), for
// the smallest calls, whose 32 x 32 tiles are fewer than the compute units: a wave's chain of matrix instructions is a quarter
// as long.  A wave's part is up to a few pieces (two at d = 256, four at 512): its whole pieces are all loaded before the first is
// multiplied, whether they fill a block of U or not (element by element, one after the other, the rest of a block cost up to 27 %
// of a call; us, element by element / so: B = 256, N = 1, d = 256 20.6 / 15.5; 512, 4, 256 22.8 / 17.9; 256, 4, 384 18.4 / 13.3).
template <bool VEC, int NW>
__global__ __launch_bounds__(64 * NW) void small_similarity_16(const float* I, const float* T, SmallShape f, float* ws) {
  __shared__ float red[NW][4][64];
  constexpr int U = 4;                                  // pieces in flight
  const int z = blockIdx.z, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, up = (lane >> 4) * 4;
  const int64_t m0 = (int64_t)blockIdx.y * 16, n0 = (int64_t)blockIdx.x * 16, m = m0 + l16, n = n0 + l16;
  const float* a = (z == 0 ? I : T) + (f.rank * f.b + (m < f.b ? m : f.b - 1)) * f.d;      // a row past the end repeats the last; its results are not stored
  const float* b = (z == 0 ? T : I) + (n < f.B ? n : f.B - 1) * f.d;
  const int pieces = (int)((f.d + 15) / 16), w = __builtin_amdgcn_readfirstlane(wave);      // dealt evenly: the shorter a wave's chain, the fewer roundings
  const int k0 = w * pieces / NW * 16, end = (w + 1) * pieces / NW * 16, k1 = end < (int)f.d ? end : (int)f.d;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int k = k0;
  for (; k + 16 * U <= k1; k += 16 * U) {
    f32x4 x[U], y[U];
#pragma unroll
    for (int c = 0; c < U; ++c) { x[c] = load4<VEC>(a, k + 16 * c + up); y[c] = load4<VEC>(b, k + 16 * c + up); }
#pragma unroll
    for (int c = 0; c < U; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c][e], y[c][e], acc, 0, 0, 0);
  }
  if (k < k1) {                                         // up to U - 1 whole pieces more
    const int left = (k1 - k) / 16;
    f32x4 x[U - 1], y[U - 1];
#pragma unroll
    for (int c = 0; c < U - 1; ++c)
      if (c < left) { x[c] = load4<VEC>(a, k + 16 * c + up); y[c] = load4<VEC>(b, k + 16 * c + up); }
#pragma unroll
    for (int c = 0; c < U - 1; ++c)
      if (c < left) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c][e], y[c][e], acc, 0, 0, 0);
      }
    k += 16 * left;
    if (k < k1) {                                       // the last piece, element by element: past k1 both operands count as 0
      float u[4], v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int kk = k + up + e, kc = kk < k1 ? kk : k1 - 1;
        u[e] = kk < k1 ? a[kc] : 0.f;
        v[e] = kk < k1 ? b[kc] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e], v[e], acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  if (wave >= 4) return;                                // wave r: the rows 4 (lane / 16) + r
  float v = red[0][wave][lane];
#pragma unroll
  for (int q = 1; q < NW; ++q) v += red[q][wave][lane];
  const int64_t row = m0 + up + wave, col = n0 + l16;
  if (row < f.b && col < f.B) ws[((size_t)z * f.b + row) * f.pitch + col] = v;
}

// Workgroup 0 adds up loss and d/ds; the others take gradient tiles (row tile, column tile, block z = whose key side):
// rows [m0, m0 + 32 R) of gT (z = 0) or gI (z = 1), key side of block z plus, in the rank's own rows, the query side of
// the other block (of the same one for the two-view loss).  The row tiles start at the rank's own rows, whose
// reduction is the longest.
template <bool WVEC, int R, int NW>
__global__ __launch_bounds__(64 * NW) void small_grads(const float* I, const float* T, SmallShape f, const float* ws, float cs, float c,
                                                       const float* row_ce, const float* row_ds, float* loss, float* gs, float* gI, float* gT) {
  __shared__ float red[NW][R * R * 16][64];
  if (blockIdx.x == 0) {
    small_scalars<NW>(f, c, row_ce, row_ds, loss, gs, &red[0][0][0]);
    return;
  }
  const int nM = (int)((f.B + 32 * R - 1) / (32 * R)), nN = (int)((f.d + 32 * R - 1) / (32 * R));
  const int w = blockIdx.x - 1, r0 = f.rank * (int)f.b;
  // tiles of all blocks in order of their distance from the own rows
  const int mt_rel = w / (nN * f.nb), rest = w - mt_rel * nN * f.nb, z = rest / nN;
  const int mt = (mt_rel + r0 / (32 * R)) % nM;
  const int64_t m0 = (int64_t)mt * 32 * R, n0 = (int64_t)(rest % nN) * 32 * R;
  f32x16 acc[R][R];
  clear(acc);
  int64_t k0, k1;
  wave_range<NW>(f.b, k0, k1);
  wave_product<R>(acc, k0, k1, AcrossK<R>(ws + (size_t)z * f.b * f.pitch, f.pitch, m0, f.B),
                  AcrossK<R>((z == 0 ? I : T) + (int64_t)r0 * f.d, f.d, n0, f.d));
  if (m0 < r0 + f.b && m0 + 32 * R > r0) {
    const int zq = f.nb == 1 ? 0 : 1 - z;
    wave_range<NW>(f.B, k0, k1);
    wave_product<R>(acc, k0, k1, OwnRows<WVEC, R>(ws + (size_t)zq * f.b * f.pitch, f.pitch, m0 - r0, f.b),
                    AcrossK<R>(zq == 0 ? T : I, f.d, n0, f.d));
  }
  float* out = z == 0 ? gT : gI;
  join_waves<R, NW>(acc, red, [&](int r, int col, float v) {
    if (m0 + r >= f.B || n0 + col >= f.d) return;
    float* p = out + (m0 + r) * f.d + n0 + col;
    *p = (f.accumulate ? *p : 0.f) + cs * v;
  });
}

// ---- bf16 features: the same two launches on the bf16 matrix instruction (32 x 32 x 16), tiles of 64 or 32 x 64.  A similarity
// is one product, exact in the instruction; a gradient entry, fp32 against bf16, is three: the fp32 value is split in
// registers into three bf16 planes that add up to it (split3_block; entries below about 2^-109 lose the last one to bf16's
// range), so nothing else is rounded that the fp32 instruction would not round.  Per 16 of the reduction that is 96 or 384 matrix cycles of a wave against 2048.
// A lane supplies 8 consecutive reduction indices (lane / 32 picks which 8 of the 16) of row 2 (lane % 32) + u of row
// block u: the two blocks' rows are interleaved, so that two neighbouring rows of an operand stored across the
// reduction come with one load.
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) float f32x8;

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// The low or the high halves of eight dwords.
__device__ __forceinline__ bf16x8 halves(const uint32_t (&w)[8], bool high) {
  u32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    r[e] = high ? __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x07060302u) : __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x05040100u);
  return __builtin_bit_cast(bf16x8, r);
}
// v = p[0] + p[1] + p[2].  (Gradient entries lie in [-1, 1] or are NaN: no plane overflows.)
__device__ __forceinline__ void split3_block(const f32x8& v, bf16x8 (&p)[3]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    p[0][e] = (__bf16)v[e];
    const float r1 = v[e] - (float)p[0][e];
    p[1][e] = (__bf16)r1;
    p[2][e] = (__bf16)(r1 - (float)p[1][e]);
  }
}

// Eight consecutive features from element idx on, in pieces of PIECE elements (8, 4 or 1: what the row pitch and the matrix's
// address allow).
template <int PIECE>
__device__ __forceinline__ bf16x8 load_row8(const uint16_t* p) {
  u32x4 w;
  if constexpr (PIECE == 8) {
    w = *reinterpret_cast<const u32x4*>(p);
  } else if constexpr (PIECE == 4) {
    const u32x2 lo = *reinterpret_cast<const u32x2*>(p), hi = *reinterpret_cast<const u32x2*>(p + 4);
    w = u32x4{lo[0], lo[1], hi[0], hi[1]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (uint32_t)p[2 * e] | (uint32_t)p[2 * e + 1] << 16;
  }
  return __builtin_bit_cast(bf16x8, w);
}
// The same where only `n` (1 to 8; at most 0: none) of the eight exist, zeros behind them.
__device__ __forceinline__ bf16x8 load_row8_part(const uint16_t* p, int n) {
  u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e < n) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
  return __builtin_bit_cast(bf16x8, w);
}

// This wave's part of a reduction of length K, in 16-deep pieces dealt in runs.
template <int NW>
__device__ __forceinline__ void wave_range16(int K, int& k0, int& k1) {
  const int per = ((K + 15) / 16 + NW - 1) / NW * 16;
  k0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * per;
  k1 = k0 + per < K ? k0 + per : K;
}

// Adds up the waves' partial 32 RB x 64 tiles in a fixed order, through red (NW / 2 tiles): the upper half of the waves hands
// its sums to the lower, whose sums are then added in wave order.  out(row, column, two values): an even column and the next, which
// a lane hands on together so that a half-wave stores whole lines.
template <int RB, int NW, class FOut>
__device__ __forceinline__ void join_waves_64(f32x16 (&acc)[RB][2], float (*red)[32 * RB][64], FOut out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto put = [&](int w) {
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[w][(u * 2 + v) * 16 + r][lane] = acc[u][v][r];
  };
  if (wave >= NW / 2) put(wave - NW / 2);
  __syncthreads();
  if (wave < NW / 2) {
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][v][r] += red[wave][(u * 2 + v) * 16 + r][lane];
    put(wave);                                          // (each lane rewrites what it alone has just read)
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16 * RB / NW; ++q) {
    const int ur = q * NW + wave, u = ur >> 4, r = ur & 15, idx = u * 32 + r;
    f32x2 s = {red[0][idx][lane], red[0][idx + 16][lane]};
#pragma unroll
    for (int w = 1; w < NW / 2; ++w) {
      s[0] += red[w][idx][lane];
      s[1] += red[w][idx + 16][lane];
    }
    out(RB * ((r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) + u, 2 * (lane & 31), s);
  }
}

// STREAM: the similarities are written past the caches (see stream_similarities).
template <int PIECE, int RB, int NW, bool STREAM>
__global__ __launch_bounds__(64 * NW) void small_similarity_bf16(const uint16_t* I, const uint16_t* T, SmallShape f, float* ws) {
  __shared__ float red[NW / 2][32 * RB][64];
  const int z = blockIdx.z, l32 = threadIdx.x & 31, up = upper_half() * 8, d = (int)f.d;
  const int64_t m0 = (int64_t)blockIdx.y * 32 * RB, n0 = (int64_t)blockIdx.x * 64;
  const uint16_t* X = (z == 0 ? I : T) + f.rank * f.b * f.d;
  const uint16_t* Y = z == 0 ? T : I;
  const uint16_t *a[RB], *b[2];                         // a row past the end repeats the last; its results are not stored
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int64_t m = m0 + RB * l32 + u;
    a[u] = X + (m < f.b ? m : f.b - 1) * f.d + up;
  }
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int64_t n = n0 + 2 * l32 + v;
    b[v] = Y + (n < f.B ? n : f.B - 1) * f.d + up;
  }
  f32x16 acc[RB][2];
  clear(acc);
  int k0, k1;
  wave_range16<NW>(d, k0, k1);
  // one 16-deep piece of both operands
  struct Piece { bf16x8 x[RB], y[2]; };
  auto product = [&](const Piece& p) {
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) acc[u][v] = mfma_bf16(p.x[u], p.y[v], acc[u][v]);
  };
  auto fetch = [&](Piece& p, int k) {
#pragma unroll
    for (int u = 0; u < RB; ++u) p.x[u] = load_row8<PIECE>(a[u] + k);
#pragma unroll
    for (int v = 0; v < 2; ++v) p.y[v] = load_row8<PIECE>(b[v] + k);
  };
  int k = k0;
  for (; k + 64 <= k1; k += 64) {                       // four pieces in flight
    Piece p[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) fetch(p[c], k + 16 * c);
#pragma unroll
    for (int c = 0; c < 4; ++c) product(p[c]);
  }
  const int whole = k < k1 ? (k1 - k) / 16 : 0;         // up to three more, all loaded before the first is multiplied
  {
    Piece p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (c < whole) fetch(p[c], k + 16 * c);
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (c < whole) product(p[c]);
  }
  k += 16 * whole;
  if (k < k1) {
    const int n = k1 - k - up;
    Piece p;
#pragma unroll
    for (int u = 0; u < RB; ++u) p.x[u] = load_row8_part(a[u] + k, n);
#pragma unroll
    for (int v = 0; v < 2; ++v) p.y[v] = load_row8_part(b[v] + k, n);
    product(p);
  }
  float* W = ws + (size_t)z * f.b * f.pitch;
  join_waves_64<RB, NW>(acc, red, [&](int r, int c, const f32x2& v) {
    if (m0 + r >= f.b || n0 + c >= f.B) return;
    float* p = W + (m0 + r) * f.pitch + n0 + c;
    if (f.pitch % 4 == 0) {                                // (what lies in the pitch behind a row is free)
      if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x2*>(p));
      else *reinterpret_cast<f32x2*>(p) = v;
    } else {
      p[0] = v[0];
      if (n0 + c + 1 < f.B) p[1] = v[1];
    }
  });
}

// Two neighbouring features of one row, from an even column of a matrix of even width on a 4-byte boundary (PAIR), or one by
// one (next: 0 where the second does not exist, the first is then repeated).
template <bool PAIR>
__device__ __forceinline__ uint32_t load_feature_pair(const uint16_t* p, int next) {
  if constexpr (PAIR) return *reinterpret_cast<const uint32_t*>(p);
  return (uint32_t)p[0] | (uint32_t)p[next] << 16;
}

// As small_grads, on tiles of 32 RB x 64.  PAIR: see load_feature_pair.  WVEC: the matrices' pitch is a multiple of 4 floats.  RB = 1 with
// 16 waves (flat_gradients) against RB = 2 with 8: B = 1024, N = 2, d = 256 20.0 -> 13.1 us of a call's 31.1 -> 23.6.  In those 13.1 the query side of the
// own rows costs 5.7, the key side 3.1 and cutting the entries into planes 1.5; one list of both sides' pieces, four in flight, was no faster, nor
// 16 x 16 x 32 products, which touch half the cache lines.
template <bool PAIR, bool WVEC, int RB, int NW>
__global__ __launch_bounds__(64 * NW) void small_grads_bf16(const uint16_t* I, const uint16_t* T, SmallShape f, const float* ws, float cs, float c,
                                                            const float* row_ce, const float* row_ds, float* loss, float* gs, float* gI, float* gT) {
  constexpr int ROWS = 32 * RB, AHEAD = RB == 2 ? 3 : 2;
  __shared__ float red[NW / 2][ROWS][64];
  if (blockIdx.x == 0) {
    small_scalars<NW>(f, c, row_ce, row_ds, loss, gs, &red[0][0][0]);
    return;
  }
  const int nM = (int)((f.B + ROWS - 1) / ROWS), nN = (int)((f.d + 63) / 64), r0 = f.rank * (int)f.b, d = (int)f.d;
  const int w = blockIdx.x - 1, mt_rel = w / (nN * f.nb), rest = w - mt_rel * nN * f.nb, z = rest / nN;
  const int mt = (mt_rel + r0 / ROWS) % nM;             // the longest reductions, those of the own rows, first
  const int m0 = mt * ROWS, n0 = (rest % nN) * 64;
  const int l32 = threadIdx.x & 31, l2 = 2 * l32, up = upper_half() * 8;
  const int n = n0 + l2 < d ? n0 + l2 : (d - 1) & ~1, next = n + 1 < d ? 1 : 0;     // columns n, n + 1 of this lane
  f32x16 acc[RB][2];
  clear(acc);
  // One 16-deep piece of a reduction as it comes from memory: this lane's 8 gradient entries of either row block and its 8 pairs
  // of features.  PART: only the indices below lim exist; the features of the others repeat the last one's, their
  // gradient entries count as 0.
  struct Raw { f32x8 g[RB]; uint32_t q[8]; };
  auto features = [&](Raw& t, const uint16_t* M, int k, int lim, auto part) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = !decltype(part)::value || k + up + e < lim ? k + e : lim - 1 - up;
      t.q[e] = load_feature_pair<PAIR>(M + (int64_t)kk * d, next);
    }
  };
  auto consume = [&](const Raw& t) {
    const bf16x8 y[2] = {halves(t.q, false), halves(t.q, true)};
    bf16x8 x[RB][3];
#pragma unroll
    for (int u = 0; u < RB; ++u) split3_block(t.g[u], x[u]);
#pragma unroll
    for (int q = 2; q >= 0; --q)
#pragma unroll
      for (int u = 0; u < RB; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = mfma_bf16(x[u][q], y[v], acc[u][v]);
  };
  // the pieces of [k0, k1), each fetched AHEAD - 1 before its use
  auto reduce = [&](int K, auto fetch) {
    int k0, k1;
    wave_range16<NW>(K, k0, k1);
    const int full = k0 < k1 ? (k1 - k0) / 16 : 0;
    Raw t[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD - 1; ++u)
      if (u < full) fetch(t[u], k0 + 16 * u, k1, std::false_type{});
    int i = 0;
    for (; i + AHEAD <= full; i += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (i + u + AHEAD - 1 < full) fetch(t[(u + AHEAD - 1) % AHEAD], k0 + 16 * (i + u + AHEAD - 1), k1, std::false_type{});
        consume(t[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD - 1; ++u)
      if (i + u < full) consume(t[u]);
    if (k0 + 16 * full < k1) {
      fetch(t[0], k0 + 16 * full, k1, std::true_type{});
      consume(t[0]);
    }
  };
  {                                                     // key side: G[k][m] down the rank's rows
    const int m = m0 + RB * l32 < f.B ? m0 + RB * l32 : RB == 2 ? (int)(f.B - 1) & ~1 : (int)f.B - 1, mnext = m + 1 < f.B ? 1 : 0;
    const float* G = ws + (size_t)z * f.b * f.pitch + up * f.pitch + m;
    const uint16_t* X = (z == 0 ? I : T) + (int64_t)(r0 + up) * d + n;
    reduce((int)f.b, [&](Raw& t, int k, int lim, auto part) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool in = !decltype(part)::value || k + up + e < lim;
        const float* p = G + (int64_t)(in ? k + e : lim - 1 - up) * f.pitch;
        f32x2 v;
        if constexpr (RB == 1) v[0] = p[0];
        else if constexpr (WVEC) v = *reinterpret_cast<const f32x2*>(p);     // (what lies in the pitch behind a row feeds no stored entry)
        else v = f32x2{p[0], p[mnext]};
#pragma unroll
        for (int u = 0; u < RB; ++u) t.g[u][e] = in ? v[u] : 0.f;
      }
      features(t, X, k, lim, part);
    });
  }
  if (m0 < r0 + f.b && m0 + ROWS > r0) {                // query side of the own rows: G[m][k] along all rows
    const int zq = f.nb == 1 ? 0 : 1 - z;
    const float* G[RB];
    bool own[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int64_t i = m0 + RB * l32 + u - r0;
      own[u] = i >= 0 && i < f.b;
      G[u] = ws + (size_t)zq * f.b * f.pitch + (own[u] ? i : 0) * f.pitch + up;
    }
    const uint16_t* Y = (zq == 0 ? T : I) + (int64_t)up * d + n;
    reduce((int)f.B, [&](Raw& t, int k, int lim, auto part) {
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        if constexpr (WVEC && !decltype(part)::value) {
          const f32x4 lo = *reinterpret_cast<const f32x4*>(G[u] + k), hi = *reinterpret_cast<const f32x4*>(G[u] + k + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) { t.g[u][e] = own[u] ? lo[e] : 0.f; t.g[u][4 + e] = own[u] ? hi[e] : 0.f; }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bool in = !decltype(part)::value || k + up + e < lim;
            const float v = G[u][in ? k + e : lim - 1 - up];
            t.g[u][e] = own[u] && in ? v : 0.f;
          }
        }
      }
      features(t, Y, k, lim, part);
    });
  }
  float* out = z == 0 ? gT : gI;
  join_waves_64<RB, NW>(acc, red, [&](int r, int col, const f32x2& v) {
    if (m0 + r >= f.B || n0 + col >= d) return;
    float* p = out + (int64_t)(m0 + r) * d + n0 + col;
    if (f.out_pairs) {
      f32x2 o = {0.f, 0.f};
      if (f.accumulate) o = *reinterpret_cast<f32x2*>(p);
      *reinterpret_cast<f32x2*>(p) = f32x2{o[0] + cs * v[0], o[1] + cs * v[1]};
    } else {
      p[0] = (f.accumulate ? p[0] : 0.f) + cs * v[0];
      if (n0 + col + 1 < d) p[1] = (f.accumulate ? p[1] : 0.f) + cs * v[1];
    }
  });
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

namespace {

// Up to this many 32 x 32 similarity tiles: 16 x 16 ones.  (us a call, 32 / 16.  At 32 tiles, B = 256, N = 4: d = 16 11.7 / 11.5,
// 128 15.4 / 12.4, 256 13.8 / 12.8, 512 16.0 / 13.7, 768 18.2 / 14.8.  At 128, B = 512, N = 4: 15.5 / 15.3, 19.7 / 17.1, 18.0 / 17.9,
// 21.2 / 20.6, 27.6 / 26.5.  At 170, B = 544, N = 4: 17.5 / 17.5, 21.7 / 19.4, 20.0 / 20.5, 25.3 / 26.2, 33.3 / 34.7.  At 256, B = 512,
// N = 2: 16.1 / 16.4, 20.7 / 18.9, 18.5 / 20.0, 25.1 / 27.7, 33.4 / 37.4.)
constexpr int64_t SIM16_MOST = 128;

// bf16 features: similarities written past the caches, or kept in them for the softmax?  Up to 32 MiB fit the eight L2s, where they
// would sit dirty until the kernel's end writes them back; up to 256 MiB stay in the last-level cache; more does not.  (Streamed /
// plain, us a call: 4 MiB, B = 1024, N = 2, d = 256: 34.3 / 35.0; 8 MiB, 1024, 1, 100: 43.9 / 45.0; 16 MiB, 2048, 2, 256: 60.8 / 63.8;
// 25 MiB, 2560, 2, 100: 85.7 / 85.0; 32 MiB, 4096, 4, 100: 94.6 / 95.5; 2048, 1, 256: 88.6 / 89.2; 40 MiB, 2304, 1, 100: 102.8 / 101.4;
// 78 MiB, 3200, 1, 100: 156 / 151; 128 MiB, 4096, 1, 100: 223 / 217; 200 MiB, 5120, 1, 100: 407 / 405; 312 MiB, 6400, 1, 100: 613 / 630;
// 512 MiB, 8192, 1, 100: 939 / 978.)
bool stream_similarities(size_t bytes) { return bytes <= ((size_t)32 << 20) || bytes > ((size_t)256 << 20); }

size_t matrix_bytes(size_t nb, int64_t b, int64_t pitch) { return align_up(nb * b * pitch * sizeof(float)); }
size_t lean_bytes(size_t nb, int64_t b, int64_t pitch) { return matrix_bytes(nb, b, pitch) + 2 * align_up(nb * b * sizeof(float)); }

// Floats between the rows of a block's matrix: whole 16-byte pieces, except where that alone would take a call out of the
// static scratch array.
int64_t row_pitch(int64_t b, int64_t B, size_t nb) {
  const int64_t padded = (B + 3) / 4 * 4;
  return lean_bytes(nb, b, padded) > DISCO_STATIC_SCRATCH_BYTES && lean_bytes(nb, b, B) <= DISCO_STATIC_SCRATCH_BYTES ? B : padded;
}

// bf16 features: tiles of half the rows by twice the waves (32 x 64, 8 waves a similarity tile, 16 a gradient tile), or 64 x 64?  Half as long
// a chain per wave and twice the workgroups, each with the same launch and the same sum over its waves.  Gradients: for the rank's own rows,
// whose reduction (b + B) is the longest, if their tiles leave every other compute unit idle, and unless the tiles of the
// other rows, whose reduction is short, are so many that what they have in common outweighs it.  (us a call, 64 rows / 32; b, N, d: 32, 16, 768
// 21.2 / 19.5; 464, 1, 500 28.0 / 23.1; 512, 2, 256 34.2 / 27.7; 88, 32, 300 52.5 / 39.9; 968, 2, 200 66.4 / 60.2; 274, 32, 200 140 / 103; own tiles
// 132 and more: 2056, 2, 77 180 / 209; 2274, 1, 100 107 / 117; 312, 1, 1000 27.3 / 30.2; 684, 2, 512 53.6 / 56.5; 1317, 2, 200 104 / 110; many others: 68, 32, 1024 48.5 / 52.9; 100, 32, 1000 65 / 77;
// 198, 16, 768 66 / 78; near the line: 178, 32, 1000 two views 99 / 90; 363, 4, 500 47.6 / 45.1; 396, 2, 1000 46.4 / 44.8.)
bool flat_gradients(int64_t b, int64_t B, int64_t d, int nb) {
  const int64_t all = nb * (int64_t)cdiv(B, 64) * cdiv(d, 64), own = nb * (int64_t)cdiv(b, 64) * cdiv(d, 64);
  return own <= 128 && (all <= 256 || 3.3 * all < b + B);
}
// Similarities: while 64 x 64 tiles are fewer than half the compute units, or two to a unit where the width is few pieces.  (133, 2, 1000 25.0 / 21.6;
// 73, 4, 1024 23.7 / 20.8; 180, 4, 500 27.1 / 25.5; 96, 4, 192 19.0 / 17.5; 287, 8, 256 54.1 / 53.0; but 365, 2, 1000 42.7 / 43.4; 396, 2, 1000
// 46.4 / 48.6; 684, 2, 512 53.6 / 56.6.)
bool flat_similarities(int64_t b, int64_t B, int64_t d, int nb) {
  const int64_t all = nb * (int64_t)cdiv(b, 64) * cdiv(B, 64);
  return all <= 128 || (all <= 512 && d <= 256);
}

// Estimated time of the small kernels: launches, products at the rate they reach (fp32 features 85 TFLOP/s, bf16 ones 200; less
// where rows are not whole pieces), and the longest reduction that the waves of one workgroup walk (a tile of the rank's
// own gradient rows).  bf16 features on gradient tiles of 32 rows: a fit (6 % rms over 40 calls of 13 to 74 us of whole 64-column tiles, within
// 0.92 to 1.2 of most others').
double small_rate_us(int64_t b, int64_t B, int64_t d, int dtype, int nb, bool flat) {
  if (flat) {
    const double us = (4.5 + 0.0118 * d) * 1e-6 * nb * b * B + 0.004 * (b + B) + 0.0193 * nb * cdiv(B, 64) * cdiv(d, 64);
    return 12.3 + us * (d % 2 ? 1.7 : d % 64 ? 1.2 : 1.0);
  }
  if (dtype == DISCO_BF16) return 14.0 + 0.5 * nb * (double)b * B * d * (d % 2 ? 1.5 : 1.0) * 12.0 / 200e6 + 1.15 * (b + B) / 128;
  const double macs = 0.5 * nb * (double)b * B * d, slow = d % 4 ? 1.9 : 1.0;
  const bool big = (double)nb * cdiv(B, 64) * cdiv(d, 64) >= 256;
  const double chain = (b + B) * (big ? 32.0 * 4 / 4 : 32.0 / 8) / 2200.0;
  return 14.0 + slow * macs * 12.0 / 85e6 + chain;
}

// Rows of reduction that the busiest compute unit walks in the gradient kernel on T x T tiles, one workgroup to a unit: b + B in a tile
// of the rank's own rows, which come first, b in the others.
double longest_walk(int64_t T, int64_t b, int64_t B, int64_t d, int nb) {
  const double units = 256.0, all = (double)nb * cdiv(B, T) * cdiv(d, T), own = std::min(all, (double)nb * cdiv(b, T) * cdiv(d, T)), rest = all - own;
  if (all <= units) return b + B;
  if (rest < units / 8) return std::ceil(own / units) * (b + B);
  return std::max((double)(b + B), (own * (b + B) + rest * b) / units + 0.5 * (own <= units ? b : b + B));
}

// The same for narrow fp32 features, by what each kernel's slowest compute units do: their tiles are as long as wide ones', and the
// rounds of workgroups end nearly empty.
double small_walk_us(int64_t b, int64_t B, int64_t d, int nb) {
  const double pairs = 1e-6 * nb * (double)b * B, width = 1e-3 * d;
  auto rounds = [&](int64_t T) { return std::max(1.0, (double)nb * cdiv(b, T) * cdiv(B, T) / 512); };
  const bool similarity64 = (double)nb * cdiv(b, 64) * cdiv(B, 64) >= 256, grads64 = (double)nb * cdiv(B, 64) * cdiv(d, 64) >= 256;
  return 8.5 + (similarity64 ? 38.0 * rounds(64) : 10.4 * rounds(32)) * width + 3.7 * pairs +
         1e-3 * (grads64 ? 20.0 * longest_walk(64, b, B, d, nb) : 8.2 * longest_walk(32, b, B, d, nb));
}

// Against the split kernels, whose estimate is good to about 10 %: for shares of 32 rows and more of fp32 features under 128 columns
// the larger of the two estimates.  The second is a fit (8 % rms) to 800 calls of 8 to 8192 rows a share, times 0.9, so weighed that it
// moves hardly a call to split kernels that are slower.  (Measured, us, small / split, fp32 features: B = 256, N = 4, d = 512 13.5 / 48; 1024, 4,
// 512 51 / 59; 2048, 16, 128 40 / 44; 2048, 16, 512 71 / 63; and small by the first estimate alone: 4096, 16, 64 66 / 47; 2560, 1, 64 187 / 108;
// 2048, 1, 100 130 / 88; 4096, 4, 20 88 / 69.)  Other calls that the first estimate keeps on the small kernels stay there although many would
// take 0.7 of the time on the split ones (1536, 1, 200 145 / 84; bf16 2560, 1, 100 115 / 88): wider ones, bf16 features and fewer rows
// because the split kernels' gradients are further from 64 bits there (1.0 to 1.6 times the error in most, up to 6 at s = 100; on the calls
// that move at most 0.98 times, mostly 0.5 to 0.75, and of 297 drawn ones none takes longer, half 0.66 of the time or less); the path by
// name's (lean) because its split kernels take the rows in chunks.
double small_us(int64_t b, int64_t B, int64_t d, int dtype, int nb, bool lean) {
  double us = small_rate_us(b, B, d, dtype, nb, false);
  // (bf16 calls that 32-row tiles move here from the split kernels: with an allowance for the two estimates)
  if (dtype == DISCO_BF16 && !lean && flat_gradients(b, B, d, nb)) us = std::min(us, 1.15 * small_rate_us(b, B, d, dtype, nb, true));
  return lean || dtype == DISCO_BF16 || d >= 128 || b < 32 ? us : std::max(us, small_walk_us(b, B, d, nb));
}

// Workspace of the split kernels may reach this where the fp32 blocks of the small ones need less.
constexpr size_t SPLIT_LIMIT = (size_t)8 << 30;

// The split kernels' workspace where they are the faster choice, else 0.  lean_only: they keep to what the small ones take.
size_t split_bytes(int64_t B, int64_t d, int64_t b, int dtype, int nb, bool lean_only, size_t* limit) {
  const size_t lean = lean_bytes(nb, b, row_pitch(b, B, nb));
  *limit = lean_only || lean > SPLIT_LIMIT ? lean : SPLIT_LIMIT;
  if (!split_supported(B, b)) return 0;
  size_t bytes;
  const double us = split_estimate_us(B, d, b, dtype, nb, *limit, &bytes);
  return bytes && us < small_us(b, B, d, dtype, nb, lean_only) ? bytes : 0;
}

void small_run(const Problem& p) {
  SmallShape f;
  f.b = p.b; f.B = p.B; f.d = p.d; f.nb = loss_blocks(p.variant);
  f.pitch = row_pitch(p.b, p.B, f.nb);
  f.rank = p.rank; f.variant = p.variant; f.accumulate = p.accumulate;
  f.out_pairs = p.d % 2 == 0 && (reinterpret_cast<uintptr_t>(p.gI) | reinterpret_cast<uintptr_t>(p.gT)) % 8 == 0;
  const unsigned nb = (unsigned)f.nb;
  const float c = loss_norm(p.B, p.variant), cs = c * p.s;
  float* W = static_cast<float*>(p.ws);
  float* row_ce = reinterpret_cast<float*>(static_cast<char*>(p.ws) + matrix_bytes(nb, p.b, f.pitch));
  float* row_ds = reinterpret_cast<float*>(reinterpret_cast<char*>(row_ce) + align_up((size_t)nb * p.b * sizeof(float)));
  const uintptr_t address = reinterpret_cast<uintptr_t>(p.I) | reinterpret_cast<uintptr_t>(p.T);
  const bool wvec = f.pitch % 4 == 0;
  auto sim_grid = [&](int tile) { return dim3(cdiv(p.B, tile), cdiv(p.b, tile), nb); };
  auto grad_grid = [&](int tile) { return dim3(1 + nb * cdiv(p.B, tile) * cdiv(p.d, tile)); };
  auto softmax = [&] {
    stage_mark(p.stream, 1);
    auto waves = [&](auto kernel) { kernel<<<dim3(cdiv(nb * p.b, 4)), 256, 0, p.stream>>>(W, p.b, p.B, f.pitch, (int)nb, p.rank, p.s, row_ce, row_ds, p.variant); };
    if (!wvec || p.B > WAVE_ROW_COLUMNS)
      naive_row_softmax<<<dim3((unsigned)p.b, nb), 256, 0, p.stream>>>(W, p.b, p.B, f.pitch, p.rank, p.s, row_ce, row_ds, p.variant);
    else if (p.B <= 256) waves(naive_wave_softmax<1>);
    else if (p.B <= 512) waves(naive_wave_softmax<2>);
    else if (p.B <= 1024) waves(naive_wave_softmax<4>);
    else waves(naive_wave_softmax<8>);
    stage_mark(p.stream, 2);
    stage_mark(p.stream, 3);
  };
  stage_mark(p.stream, 0);
  if (p.dtype == DISCO_BF16) {
    const uint16_t* I = static_cast<const uint16_t*>(p.I);
    const uint16_t* T = static_cast<const uint16_t*>(p.T);
    const bool flat_sim = flat_similarities(p.b, p.B, p.d, nb), flat_grads = flat_gradients(p.b, p.B, p.d, nb);
    auto sim = [&](auto kernel, int rows) { kernel<<<dim3(cdiv(p.B, 64), cdiv(p.b, rows), nb), rows == 64 ? 256 : 512, 0, p.stream>>>(I, T, f, W); };
    auto similarity = [&](auto piece) {
      constexpr int P = decltype(piece)::value;
      if (flat_sim) sim(small_similarity_bf16<P, 1, 8, true>, 32);
      else if (stream_similarities(matrix_bytes(nb, p.b, f.pitch))) sim(small_similarity_bf16<P, 2, 4, true>, 64);
      else sim(small_similarity_bf16<P, 2, 4, false>, 64);
    };
    if (p.d % 8 == 0 && address % 16 == 0) similarity(std::integral_constant<int, 8>{});
    else if (p.d % 4 == 0 && address % 8 == 0) similarity(std::integral_constant<int, 4>{});
    else similarity(std::integral_constant<int, 1>{});
    softmax();
    auto go = [&](auto kernel, int rows) {
      kernel<<<dim3(1 + nb * cdiv(p.B, rows) * cdiv(p.d, 64)), rows == 64 ? 512 : 1024, 0, p.stream>>>(I, T, f, W, cs, c, row_ce, row_ds, p.loss, p.gs, p.gI, p.gT);
    };
    auto grads = [&](auto pair, auto vec) {
      constexpr bool PR = decltype(pair)::value, VC = decltype(vec)::value;
      if (flat_grads) go(small_grads_bf16<PR, VC, 1, 16>, 32);
      else go(small_grads_bf16<PR, VC, 2, 8>, 64);
    };
    const bool pair = p.d % 2 == 0 && address % 4 == 0;
    if (pair) { if (wvec) grads(std::true_type{}, std::true_type{}); else grads(std::true_type{}, std::false_type{}); }
    else { if (wvec) grads(std::false_type{}, std::true_type{}); else grads(std::false_type{}, std::false_type{}); }
  } else {
    const float* I = static_cast<const float*>(p.I);
    const float* T = static_cast<const float*>(p.T);
    const bool vec = p.d % 4 == 0 && address % 16 == 0;
    // 64 x 64 tiles (four waves) once they give every compute unit one, else 32 x 32 (eight waves)
    auto big = [&](int64_t rows, int64_t cols) { return (int64_t)nb * cdiv(rows, 64) * cdiv(cols, 64) >= 256; };
    auto sim = [&](auto kernel, int tile, int waves) { kernel<<<sim_grid(tile), 64 * waves, 0, p.stream>>>(I, T, f, W); };
    auto grads = [&](auto kernel, int tile, int waves) {
      kernel<<<grad_grid(tile), 64 * waves, 0, p.stream>>>(I, T, f, W, cs, c, row_ce, row_ds, p.loss, p.gs, p.gI, p.gT);
    };
    if (big(p.b, p.B)) { if (vec) sim(small_similarity<true, 2, 4>, 64, 4); else sim(small_similarity<false, 2, 4>, 64, 4); }
    else if ((int64_t)nb * cdiv(p.b, 32) * cdiv(p.B, 32) <= SIM16_MOST) { if (vec) sim(small_similarity_16<true, 8>, 16, 8); else sim(small_similarity_16<false, 8>, 16, 8); }
    else { if (vec) sim(small_similarity<true, 1, 8>, 32, 8); else sim(small_similarity<false, 1, 8>, 32, 8); }
    softmax();
    if (big(p.B, p.d)) { if (wvec) grads(small_grads<true, 2, 4>, 64, 4); else grads(small_grads<false, 2, 4>, 64, 4); }
    else { if (wvec) grads(small_grads<true, 1, 8>, 32, 8); else grads(small_grads<false, 1, 8>, 32, 8); }
  }
  stage_mark(p.stream, 4);
  stage_mark(p.stream, 5);
}

}  // namespace

size_t naive_workspace_bytes(int64_t B, int64_t d, int32_t N, int dtype, int variant, bool lean) {
  const int64_t b = B / N;
  const int nb = loss_blocks(variant);
  const size_t least = lean_bytes(nb, b, row_pitch(b, B, nb));
  size_t limit;
  const size_t split = split_bytes(B, d, b, dtype, nb, lean, &limit);
  return split > least ? split : least;             // (unaligned gradients take the small kernels whatever the plan)
}

void naive_describe(int64_t B, int64_t d, int32_t N, int dtype, int variant, bool lean, disco_plan* out) {
  const int64_t b = B / N;
  const int nb = loss_blocks(variant);
  size_t limit;
  if (split_bytes(B, d, b, dtype, nb, lean, &limit)) {
    split_describe(B, d, b, dtype, nb, limit, out);
    return;
  }
  out->kernels = DISCO_KERNELS_SMALL;
  out->row_chunks = out->key_panels = out->query_splits = out->key_splits = 1;
  out->microseconds = small_us(b, B, d, dtype, nb, lean);
}

// Is a call that the bf16 tile kernels take faster on the small ones?  Few tiles leave those kernels with their seven launches,
// about 21 us on top of the tiles' estimate whatever the shape; the small ones are three.  27 are allowed: within those 6 us a call
// keeps the small kernels' fp32 numerators, whose gradients are 1e-5 and more of their 2-norm nearer.  (Measured, us, tiles / small,
// bf16: B = 256, N = 1, d = 128: 29 / 14; 512, 2, 256: 29 / 17; 1024, 4, 512: 34 / 26; 1024, 2, 256: 33 / 27; 1024, 4, 1024: 44 / 33; 2048, 16,
// 512: 35 / 41; 2048, 4, 256: 35 / 51; 4096, 32, 512: 38 / 65.)
// That line is of 64-row tiles; where the gradients have 32-row ones, a call estimated 5 us faster than on the tile kernels moves too (417, 4, 128
// two views 33.6 / 29.0; 274, 8, 256 40.8 / 37.5).
bool small_beats_tiles(int64_t B, int64_t d, int32_t N, int variant) {
  const int nb = loss_blocks(variant);
  const int64_t b = B / N;
  const double tiles = mfma_stored_estimate_us(B, d, N, variant), us = small_rate_us(b, B, d, DISCO_BF16, nb, false);
  if (us < 60.0 && us < tiles + 27.0) return true;
  return flat_gradients(b, B, d, nb) && small_rate_us(b, B, d, DISCO_BF16, nb, true) < tiles + 16.0;
}

int naive_run(const Problem& p) {
  const int64_t b = p.b, B = p.B;
  const int nb = loss_blocks(p.variant);
  size_t limit;
  if (split_bytes(B, p.d, b, p.dtype, nb, p.lean, &limit) && split_aligned(p)) return split_run(p, limit);
  small_run(p);
  return hipGetLastError() == hipSuccess ? DISCO_OK : DISCO_ERR_HIP;
}

}  // namespace disco

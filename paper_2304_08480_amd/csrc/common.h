// Internal declarations shared by the host dispatch and the kernel files of libdisco.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/disco.h"

namespace disco {

// One of the two logit blocks of a rank (Sec. 4.1 Eq. 6).  Block A: X = I_r, Y = T, query-side
// gradient goes to gI rows R_r and key-side gradient to all rows of gT; block C is the mirror image.
struct Problem {
  const void* I;
  const void* T;
  int64_t B, d;
  int32_t rank, N;
  int64_t b;          // B / N
  float s;
  int dtype;
  int accumulate;
  bool lean;          // fp32 path: see naive_workspace_bytes
  size_t limit;       // bf16 paths: most bytes that the plan may take (NO_LIMIT: the caller's workspace is what the plan asks for)
  float* loss;
  float* gI;
  float* gT;
  float* gs;
  void* ws;
  size_t ws_bytes;
  hipStream_t stream;
  int variant;        // LOSS_CLIP: two blocks, label = own row.  LOSS_NTXENT: I = T = Z (one matrix, one block,
                      // gI = gT = gZ), label = the other view's row, the self-similarity is left out
};

enum { LOSS_CLIP = 0, LOSS_NTXENT = 1 };
constexpr size_t NO_LIMIT = ~(size_t)0;

// Global row of the positive of global row g, and the column that is left out of row g's softmax (-1: none).
__host__ __device__ inline int64_t label_row(int64_t g, int64_t B, int variant) {
  if (variant == LOSS_NTXENT) return g + B / 2 < B ? g + B / 2 : g - B / 2;
  return g;
}
__host__ __device__ inline int64_t masked_col(int64_t g, int variant) { return variant == LOSS_NTXENT ? g : -1; }
__host__ __device__ inline int loss_blocks(int variant) { return variant == LOSS_NTXENT ? 1 : 2; }
// Normalisation: 1/(2B) for the two directions of the CLIP loss, 1/B for the single one of the two-view loss.
__host__ __device__ inline float loss_norm(int64_t B, int variant) { return (variant == LOSS_NTXENT ? 1.0f : 0.5f) / (float)B; }

// v over the wave by f (of two floats or two ints), the same in all lanes: four steps inside 16 lanes, two between them, none through
// the LDS.  (Partners l ^ 1, l ^ 2, 7 - l, 15 - l, l ^ 16, l ^ 32.)
template <int CTRL, class V>
__device__ __forceinline__ V dpp(V v) {
  return __builtin_bit_cast(V, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <class V, class F>
__device__ __forceinline__ V wave_reduce(V v, F f) {
  static_assert(sizeof(V) == 4);
  v = f(v, dpp<0xB1>(v));
  v = f(v, dpp<0x4E>(v));
  v = f(v, dpp<0x141>(v));
  v = f(v, dpp<0x140>(v));
  const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false);
  const uint32_t p0 = p[0], p1 = p[1];
  v = f(__builtin_bit_cast(V, p0), __builtin_bit_cast(V, p1));
  const auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false);
  const uint32_t q0 = q[0], q1 = q[1];
  return f(__builtin_bit_cast(V, q0), __builtin_bit_cast(V, q1));
}

// Benchmark stage timing (see disco_set_stage_events): records events[k] on `st` if it exists.
void stage_mark(hipStream_t st, int k);
bool stage_marks_on();

// The plans of a thread's last few shapes.  Comparing a few hundred candidates takes 3 to 10 us of host time and a call
// asks for its plan two or three times (workspace check, route, launch), which a short call would wait for.
template <class Plan, int NKEY>
struct PlanCache {
  struct Entry { int64_t key[NKEY]; Plan plan; bool set = false; } entry[4];
  int next = 0;
  template <class F>
  Plan get(const int64_t (&key)[NKEY], F make) {
    for (Entry& e : entry) {
      bool same = e.set;
      for (int i = 0; i < NKEY; ++i) same = same && e.key[i] == key[i];
      if (same) return e.plan;
    }
    Entry& e = entry[next];
    next = (next + 1) % 4;
    e.plan = make();
    for (int i = 0; i < NKEY; ++i) e.key[i] = key[i];
    e.set = true;
    return e.plan;
  }
};

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

// The fp32 path.  lean: within the memory of its fp32 logit blocks (what DISCO_PATH_NAIVE by name asks for).
size_t naive_workspace_bytes(int64_t B, int64_t d, int32_t N, int dtype, int variant, bool lean);
int naive_run(const Problem& p);
bool small_beats_tiles(int64_t B, int64_t d, int32_t N, int variant);

// Its large calls (split_kernels.hip): shapes they take, gradients they can store, their estimated time and workspace with the
// workspace kept within `limit` (*bytes = 0: impossible), and the call in that plan.
bool split_supported(int64_t B, int64_t b);
bool split_aligned(const Problem& p);
double split_estimate_us(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit, size_t* bytes);
int split_run(const Problem& p, size_t limit);
void split_describe(int64_t B, int64_t d, int64_t b, int dtype, int nb, size_t limit, disco_plan* out);

// the bf16 tile kernels can take the shape (materialized path; a rank share that is not a whole number of 256-row
// tiles is rounded up to them) / the share is whole tiles (what the fused and symmetric paths need too)
bool mfma_supported(int64_t B, int64_t d, int32_t N, int dtype, int variant = LOSS_CLIP);
bool mfma_whole_tiles(int64_t B, int32_t N);
double mfma_stored_estimate_us(int64_t B, int64_t d, int32_t N, int variant);      // its tile kernels, without the launches
size_t mfma_workspace_bytes(int64_t B, int64_t d, int32_t N, int variant, bool fused, size_t limit);      // the plan's within `limit`, else more
int mfma_stored_run(const Problem& p);
int mfma_fused_run(const Problem& p);
size_t mfma_sym_workspace_bytes(int64_t B, int64_t d, size_t limit);
int mfma_sym_run(const Problem& p);      // N = 1, the CLIP loss only

// Raise the dynamic-LDS limits of all their kernels (false: HIP refused).
bool mfma_raise_lds();
bool split_raise_lds();

// What a call would run (disco_describe_plan), without the fields that api.hip fills in itself.
void naive_describe(int64_t B, int64_t d, int32_t N, int dtype, int variant, bool lean, disco_plan* out);
void mfma_describe(int64_t B, int64_t d, int32_t N, int variant, bool fused, bool sym, size_t limit, disco_plan* out);

// disco_loss_fwd_bwd with its plan kept within `limit`.
size_t loss_workspace_bytes(int64_t B, int64_t d, int32_t N, int dtype, int path, size_t limit);
int loss_call(const void* I, const void* T, int64_t B, int64_t d, int32_t rank, int32_t N, float s, int dtype, int path, int accumulate,
              float* loss, float* gI, float* gT, float* gs, void* workspace, size_t workspace_bytes, void* hip_stream, size_t limit);

}  // namespace disco

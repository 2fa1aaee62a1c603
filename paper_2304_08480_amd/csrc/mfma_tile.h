// Device-side building blocks of the bf16 MFMA path: the T x T x 64 NT tile main loop (T = 256 or 128), the operand
// tile formats and the tile store of the fp32 outputs (through LDS).  Included by mfma_kernels.hip and split_kernels.hip.
//
// Shape of the loop.  A workgroup of 8 waves (two per SIMD) owns a 256x256 output tile; each wave owns
// 128x64 of it as 8x4 MFMA 16x16x32 bf16 blocks with fp32 accumulators.  What bounds the loop is power (the chip clocks at
// 1.7-1.9 GHz in it), and the 16x16x32 form does the same multiplications with half the accumulator traffic: from registers
// alone the whole chip runs 2.00-2.12 PFLOP/s of it (k_mfma_probe) against 1.86-1.96 of 32x32x16, and a call of B = 32768, N = 8, d = 512 takes
// 752 us against 821, B = 65536, d = 768 3990 against 4395.  The reduction runs in K-steps of
// 64.  Operand tiles travel global memory -> LDS directly (buffer_load_dwordx4 ... lds): no staging
// registers, no LDS write instructions, and the data in flight lives in LDS.  K-steps are 64 wide so that
// a load instruction of a reduction-contiguous operand covers 8 rows x 128 bytes, i.e. whole cache lines
// (with 32-wide steps each line is fetched in two halves and such loads cost twice as much).
//
// A direct-to-LDS load holds its wave's instruction issue for tens of cycles (more when the memory
// pipeline is backed up), during which that wave issues no MFMA.  The loop therefore splits the loading
// between the two waves of each SIMD and staggers it by half a K-step: waves 0-3 load the A operand in the
// second quarter of a K-step, waves 4-7 the B operand in the fourth, so that one wave of every SIMD is
// always free to feed the matrix pipe.  To give those loads room, the LDS (all 160 KiB) is a ring of five
// 32 KiB units, each holding one operand of one K-step: A(kt), B(kt), A(kt+1), B(kt+1) resident or landing,
// plus one unit being refilled (see kloop).
//
// T = 128 is the same loop at half the size: 4 waves of 64 x 64, waves 0-1 loading A and 2-3 B, units of 16 KiB, so that
// two workgroups share a compute unit (80 KiB of LDS each).  It moves twice the bytes per MFMA, which the compute unit's
// load path (about 64 B/clk) cannot hide: where the chip is full a K-step of two such workgroups takes 0.6 times that of a
// 256-tile of twice their work (b = 4096, B = 32768, d = 512: 915 us a call against 730).  What it is for is
// calls whose 256-tiles leave compute units idle, whose reductions are a few K-steps, or whose feature width fills half a
// 256-tile: 34 us against 49 at b = 512, B = 1024, d = 256; 75 against 96 at b = 1550, B = 6200, d = 256.
//
// Operand tile formats in one unit (T = 256; T = 128 has half the rows or half the row length):
//   format K - the operand's reduction index is contiguous in memory (element (r,k) at base[r*ld + k]):
//              256 rows of 128 bytes, 16-byte chunks XOR-swizzled with bits 1..3 of the row so that the
//              16 consecutive rows a quarter-wave reads (same chunk) hit 16 different bank groups of the
//              64-bank LDS; fragments are read with ds_read_b128.
//   format R - the operand's row index is contiguous in memory (element (r,k) at base[k*ld + r]): 64
//              reduction rows of 512 bytes; the 32-byte group index is XOR-ed with bits 0, 1 and 3
//              of the reduction row, so the 8 reduction rows (0..3 and 8..11 of 16) that a half-wave reads at once
//              cover a 256-byte bank window exactly; fragments are read with the transposing
//              ds_read_b64_tr_b16 (two per fragment).
// A direct-to-LDS load puts lane l's 16 bytes at (wave-uniform LDS base) + 16*l, so a swizzle is applied by
// choosing which global chunk each lane fetches.
//
// FMT_KA / FMT_RA read an operand kept in memory in "atoms": 16-byte pieces holding 8 consecutive columns of one
// row, laid out by groups of 64 rows, inside a group column piece by column piece, inside a column piece row by
// row: element (r, c) at ((r / 64) * (ncols / 8) + c / 8) * 512 + (r % 64) * 8 + c % 8; `ld` = elements between
// row groups (64 * ncols).  A column piece of a row group is 1 KiB of memory, a 64 x 64 block 8 KiB, and a producer
// whose lanes hold 8 consecutive columns of 32 or 64 consecutive rows stores whole 512-byte or 1 KiB runs straight
// from registers.
//   FMT_KA reduces along the columns (a K-step is 8 column pieces of each of the tile's four row groups: four
//          contiguous 8 KiB runs, and a load instruction fetches one column piece of one row group, 1 KiB).  Its LDS
//          tile keeps that order too: column piece c of the K-step at 4096 c, inside it tile row r at 16 r; the 16
//          consecutive rows a quarter-wave reads with ds_read_b128 are 256 contiguous bytes, so no swizzle.
//   FMT_RA reduces down the rows (a K-step is one row group; the tile's 256 rows are 32 column pieces of it: one
//          contiguous 32 KiB run, and a load instruction fetches one column piece, 1 KiB).  Its LDS tile keeps that
//          order: column piece c at 1024 c, inside it reduction row kap at 16 (kap ^ 4 (c % 2)), so that the
//          8 reduction rows x 2 column pieces x 2 halves which a half-wave reads at once with ds_read_b64_tr_b16
//          cover a 256-byte bank window exactly.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace disco {
namespace tile {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) _Float16 half8;
typedef __attribute__((ext_vector_type(4))) _Float16 half4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int BK = 64;
constexpr int NUNITS = 5;
constexpr int NLD = 8;                            // load instructions per loading wave and unit

// T x T output tile: 256 (8 waves, 2 along M x 4 along N, wave tile 128 x 64) or 128 (4 waves, 2 x 2, wave tile 64 x 64)
template <int T>
struct Cfg {
  static_assert(T == 128 || T == 256);
  static constexpr int WAVES = T / 32, NTHREADS = WAVES * 64;
  static constexpr int WN = WAVES / 2;                    // waves along N; also the waves that load one operand
  static constexpr int WTM = T / 2;                       // a wave's rows of the A side (64 of the B side)
  static constexpr int NFA = WTM / 16, NFB = 4;           // its 16-row fragments of the A side and of the B side
  static constexpr int UNIT_BYTES = T * BK * 2;           // one operand, one K-step: 32 or 16 KiB
  static constexpr int SMEM_BYTES = NUNITS * UNIT_BYTES;  // the ring: all 160 KiB of the CU's LDS, or half of it
};
// acc[i][j][r] of lane l: row 16 i + 4 (l / 16) + r, column 16 j + l % 16 of the wave's tile
template <int NFA>
using Acc = f32x4[NFA][4];

// Plane products of an operand pair of PA and PB planes (PS of kloop), smallest first.  Planes 0, 1, 2 of a value carry its
// leading, middle and last 8 significand bits, so with three planes on both sides the products left out (1 x 2, 2 x 1 and
// 2 x 2) come to 2^-24 of the values' own product at most and to 2^-27.5 root mean square.
template <int PA, int PB, bool SWEEPS_ = false>
struct Planes {
  static constexpr bool HALF = false, SWEEPS = SWEEPS_;
  static_assert((PA == 1 && PB == 1) || (PA == 3 && (PB == 1 || PB == 3)));
  static constexpr int N = PA == 1 ? 1 : PB == 1 ? 3 : 6;
  // two bits per product
  static constexpr uint32_t A = PA == 1 ? 0u : PB == 1 ? (2u | 1u << 2 | 0u << 4) : (2u | 0u << 2 | 1u << 4 | 1u << 6 | 0u << 8 | 0u << 10);
  static constexpr uint32_t B = PB == 1 ? 0u : (0u | 2u << 2 | 1u << 4 | 0u << 6 | 1u << 8 | 0u << 10);
};

// The same of operands kept in fp16 planes (split_kernels.hip says what each plane holds): logits of NP planes, all four products of two, and
// gradients, whose last product has the leading planes of both sides.
template <int NP>
struct HalfLogits {
  static_assert(NP == 1 || NP == 2);
  static constexpr bool HALF = true, SWEEPS = NP == 2;
  static constexpr int N = NP * NP;
  static constexpr uint32_t A = NP == 1 ? 0u : (1u | 1u << 2), B = NP == 1 ? 0u : (1u | 1u << 4);
};
template <int NP>
struct HalfGrads {
  static_assert(NP == 1 || NP == 2);
  static constexpr bool HALF = true, SWEEPS = true;
  static constexpr int N = NP + 1;
  static constexpr uint32_t A = 1u, B = NP == 1 ? 1u : (2u | 1u << 2);
};

enum { FMT_K = 0, FMT_R = 1, FMT_KA = 2, FMT_RA = 3 };
// bytes between the LDS destinations of a wave's consecutive load instructions (FMT_KA: the wave loads the 8 column
// pieces of its row group, which lie 16 T bytes apart; else its instructions fill 8 KiB contiguously)
constexpr int lds_step(int f, int T) { return f == FMT_KA ? 16 * T : 1024; }

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int N>
__device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ---- LDS reads as opaque instructions: the compiler cannot tell which direct-to-LDS load a read depends
// on and would wait for all of them; the waits are placed by hand instead (wait_frags).
template <int OFF>
__device__ __forceinline__ u32x4 ds_read128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
template <int OFF>
__device__ __forceinline__ u32x2 ds_read64_tr(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}

// Operand fragments, 16 rows x 32 of the reduction each: half of the A side's (rows 16 i of it), all of the B side's.
template <int NH>
struct FragsA {
  u32x4 f[NH];
};
struct FragsB {
  u32x4 f[4];
};
// All LDS reads issued so far have returned; ties the registers to the wait so no MFMA moves above it.
__device__ __forceinline__ void wait_frags(FragsA<4>& a, FragsB& b) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(a.f[0]), "+v"(a.f[1]), "+v"(a.f[2]), "+v"(a.f[3]), "+v"(b.f[0]), "+v"(b.f[1]), "+v"(b.f[2]), "+v"(b.f[3])
               :
               : "memory");
}
__device__ __forceinline__ void wait_frags(FragsA<2>& a, FragsB& b) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a.f[0]), "+v"(a.f[1]), "+v"(b.f[0]), "+v"(b.f[1]), "+v"(b.f[2]), "+v"(b.f[3]) : : "memory");
}

// A pointer that is the same in every lane, handed to the compiler as scalar registers: the loads below then take
// the form scalar base + 32-bit lane offset, with no 64-bit vector address arithmetic and no vector registers for it.
__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

// The `bytes` (4 GiB) from p on (both the same in every lane) as a buffer resource: loads past them return zeros and fetch nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* p, uint32_t bytes = 0xffffffffu) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(uniform_ptr(p)), 0, bytes, 0x00020000);
}

// How much of its operands a tile may read.  Whole: all of it exists.  Bounded: rows_a of the A tile's rows (FMT_K), rows_b of the B tile's
// (FMT_K) or of the reduction's (FMT_R, whose tile starts at byte col_b of a row); none if not positive.  The loop reads zeros for
// the others, by the bounds of its buffer resources, which it sets up for every K-step in any case.  (Zero-padded copies of the operands before,
// a launch and 2 (B + b) d of 2 bytes read and written: B = 30000, N = 8, d = 512, two shares 1366 / 1335 us, smaller ragged calls up to
// 12 %: 128 / 114.  Clamping rows to the last one instead would need masks where padding meets padding.  The bounds cost the instances that take
// them 10 to 30 scalar instructions a tile; whole shares run those without.)
struct Whole { static constexpr bool ON = false; };
struct Bounded {
  static constexpr bool ON = true;
  int rows_a, rows_b;
  uint32_t col_b;
};
// Bytes that exist from where K-step kt of such an operand starts.
template <int T, int FMT>
__device__ __forceinline__ uint32_t bytes_left(int rows, uint32_t col, int64_t ld, int kt) {
  const int there = FMT == FMT_R ? rows - kt * BK : rows, most = FMT == FMT_R ? BK : T;
  const uint32_t n = (uint32_t)(there < 0 ? 0 : there > most ? most : there) * (uint32_t)(ld * 2), skip = FMT == FMT_R ? col : (uint32_t)kt * (BK * 2);
  return __builtin_amdgcn_readfirstlane(FMT == FMT_K || FMT == FMT_R ? (n > skip ? n - skip : 0u) : 0xffffffffu);
}

// Rows of the reduction may carry a factor: of the B operand (FMT_R, fp16 planes), row k is multiplied by 2^-(shift[k] - least), at most by 1 and at
// least by 2^-48, when its 64-deep piece has come and before the barrier hands it on.  In the LDS, by the lanes that loaded it: each 16-byte
// piece there is one row's, so a lane's factors are its own and nothing else of the loop changes; fp16 ends at 2^-24, so a factor is taken in
// two halves.  (A copy of the operand made by a launch of its own cost every call 7 us of 201, B = 8192, N = 8, d = 512, mostly for finding nothing to do.)
struct Unshifted { static constexpr bool ON = false; };
struct RowShifts {
  static constexpr bool ON = true;
  const uint8_t* shift;   // 16-byte aligned; memory that the kernel does not write
  int least;
};
// 2^-k as fp16, 0 <= k <= 24
__device__ __forceinline__ _Float16 half_power(int k) { return __builtin_bit_cast(_Float16, (uint16_t)(k < 15 ? (15 - k) << 10 : 1 << (24 - k))); }

// The exponents of the rows of piece `piece` that loading wave lw has, 16 (T = 256) or 32 consecutive ones (scalar loads), and their use on what
// it has loaded into the unit at `lds`.
template <int T>
struct Exponents { u32x4 v[256 / T]; };
template <int T>
__device__ __forceinline__ Exponents<T> fetch_exponents(const RowShifts& s, int piece, int lw) {
  typedef const __attribute__((address_space(4))) u32x4* from;
  const uint64_t at = reinterpret_cast<uint64_t>(uniform_ptr(s.shift + piece * BK + lw * (4096 / T)));
  Exponents<T> e;
#pragma unroll
  for (int i = 0; i < 256 / T; ++i) e.v[i] = reinterpret_cast<from>(at)[i];
  return e;
}
template <int T>
__device__ __forceinline__ void shift_rows(const Exponents<T>& e, int least, char* lds, int lw, int lane) {
  // the n-th load instruction brings 64 / PPR rows, PPR = T / 8 pieces each (Operand::init)
  const int mine = lane / (T / 8) * 8;
  half8* at = reinterpret_cast<half8*>(lds + NLD * lw * 1024 + lane * 16);
#pragma unroll
  for (int h = 0; h < NLD; h += 4) {
    half8 v[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) v[n] = at[(h + n) * 64];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int byte = (h + n) * (512 / T), below = (int)(e.v[byte / 16][byte % 16 / 4] >> (byte % 4 * 8 + mine) & 255u) - least;
      const int k = below < 0 ? 0 : below < 48 ? below : 48;
      at[(h + n) * 64] = v[n] * half_power(k / 2) * half_power(k - k / 2);
    }
  }
}

// format R: what the 32-byte group index of reduction row kap is XOR-ed with
__device__ __forceinline__ int swizzle_r(int kap) { return (kap & 3) << 1 | (kap >> 3 & 1); }

// ---- per-lane addressing of one operand of a T x T tile
template <int T, int FMT, int NFRAG>
struct Operand {
  static constexpr int NRD = FMT == FMT_R ? NFRAG : FMT == FMT_KA ? 1 : 2;
  uint32_t ld_off[NLD];     // byte offset of this lane's global chunk for the wave's load instructions
  uint32_t rd[NRD];         // FMT_K: base for the K-step's first and second half; FMT_KA: base; FMT_R: base of fragment i; FMT_RA:
                            // base of the fragment's first and second transposing read
  uint32_t lds_q;           // LDS byte offset (inside the operand tile) of the wave's first load instruction

  // lw: index of this wave among the T / 64 that load this operand; row0: first tile row of this
  // wave's fragments (multiple of 64, of 128 for eight of them); ld in elements; nvalid: tile rows that exist in memory (a multiple of
  // 8, at most T): loads of the rows past them are redirected to the last existing rows, so that they
  // stay in bounds (the caller does not use the output rows or columns they feed)
  __device__ __forceinline__ void init(int64_t ld, int lw, int lane, int row0, int nvalid = T) {
    const int wave = lw;
    lds_q = FMT == FMT_KA ? wave * 1024 : NLD * wave * 1024;
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
      const int q = NLD * wave + n;               // which 1 KiB slice of the operand's unit
      if (FMT == FMT_K) {
        const int rho = 8 * q + (lane >> 3), pc = lane & 7;
        const int ch = (pc ^ ((rho >> 1) & 7)) << 3;
        const int rsrc = rho < nvalid ? rho : nvalid - 1;
        ld_off[n] = (uint32_t)(((int64_t)rsrc * ld + ch) * 2);
      } else if (FMT == FMT_KA) {                   // row group `wave`, column piece n of the K-step, row `lane` of the group
        ld_off[n] = (uint32_t)(((int64_t)wave * ld + n * 512 + lane * 8) * 2);
      } else if (FMT == FMT_RA) {
        const int c = q;                            // this instruction's column piece; lane = position in it
        ld_off[n] = (uint32_t)((c * 512 + (lane ^ ((c & 1) << 2)) * 8) * 2);
      } else {
        constexpr int PPR = T / 8;                  // 16-byte pieces per reduction row of the unit
        const int kap = (64 / PPR) * q + lane / PPR, pcw = lane % PPR;
        const int c0 = (((pcw >> 1) ^ swizzle_r(kap)) << 1) | (pcw & 1);
        const int c = (c0 << 3) < nvalid ? c0 : (nvalid >> 3) - 1;
        ld_off[n] = (uint32_t)(((int64_t)kap * ld + (c << 3)) * 2);
      }
    }
    // lane l supplies the 8 reduction indices 8 (l / 16) .. of row l % 16 of a fragment; for a transposing read it names 4
    // rows' worth (`piece`) of one reduction row and receives 4 reduction indices of its own row
    const int grp = lane >> 4, L = lane & 15;
    if (FMT == FMT_K) {
      const int row = row0 + L, g = (row >> 1) & 7;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) rd[ks] = (uint32_t)(row * 128 + (((ks * 4 + grp) ^ g) << 4));
    } else if (FMT == FMT_KA) {
      rd[0] = (uint32_t)(grp * (16 * T) + (row0 + L) * 16);
    } else if (FMT == FMT_RA) {
      const int piece = L & 3, c = (row0 >> 3) + (piece >> 1);       // + 2 per fragment: c % 2 unchanged
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int kap = grp * 8 + (L >> 2) + 4 * h;                  // + 32 ks: bit 2 unchanged
        rd[h] = (uint32_t)(c * 1024 + ((kap ^ ((c & 1) << 2)) << 4) + (piece & 1) * 8);
      }
    } else {
      const int kap = grp * 8 + (L >> 2);         // + 32 ks + 4 h: the swizzle's bits unchanged
#pragma unroll
      for (int i = 0; i < NFRAG; ++i) {
        const int G = (row0 >> 4) + i;
        rd[i] = (uint32_t)(kap * (2 * T) + ((G ^ swizzle_r(kap)) << 5) + 8 * (L & 3));
      }
    }
  }
  // this wave's n-th load instruction of the K-step whose tile starts at `base`, into the unit at `lds`.  (The buffer form: scalar
  // base + 32-bit lane offset.  Of a plain pointer the compiler keeps the offsets as 64-bit pairs where the tile loop runs more
  // than once, 32 registers in the logit kernels, and adds the base in vector registers.)
  __device__ __forceinline__ void load(int n, __amdgpu_buffer_rsrc_t base, char* lds) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(base, (__attribute__((address_space(3))) void*)(lds + __builtin_amdgcn_readfirstlane(lds_q) + n * lds_step(FMT, T)),
                                             16, ld_off[n], 0, 0, 0);
  }
  __device__ __forceinline__ void load_all(__amdgpu_buffer_rsrc_t base, char* lds) const {
#pragma unroll
    for (int n = 0; n < NLD; ++n) load(n, base, lds);
  }
};

__device__ __forceinline__ u32x4 join(u32x2 lo, u32x2 hi) { return u32x4{lo[0], lo[1], hi[0], hi[1]}; }

// fragment I of the K-step's half KS from the operand tile at LDS byte address `tile`
template <int KS, int I, int T, int FMT, int NFRAG>
__device__ __forceinline__ u32x4 read_frag(const Operand<T, FMT, NFRAG>& op, uint32_t tile) {
  if constexpr (FMT == FMT_K) return ds_read128<I * 2048>(tile + op.rd[KS]);
  else if constexpr (FMT == FMT_KA) return ds_read128<KS * 64 * T + I * 256>(tile + op.rd[0]);
  else if constexpr (FMT == FMT_RA) return join(ds_read64_tr<KS * 512 + I * 2048>(tile + op.rd[0]), ds_read64_tr<KS * 512 + I * 2048>(tile + op.rd[1]));
  else return join(ds_read64_tr<KS * 64 * T>(tile + op.rd[I]), ds_read64_tr<KS * 64 * T + 8 * T>(tile + op.rd[I]));
}
// fragments of half H (rows) of the A side, of the B side's fragments J and J + 1
template <int KS, int H, int NH, int T, int FMT>
__device__ __forceinline__ void read_a(FragsA<NH>& a, const Operand<T, FMT, 2 * NH>& op, uint32_t tile) {
  a.f[0] = read_frag<KS, H * NH>(op, tile);
  a.f[1] = read_frag<KS, H * NH + 1>(op, tile);
  if constexpr (NH == 4) {
    a.f[2] = read_frag<KS, H * NH + 2>(op, tile);
    a.f[3] = read_frag<KS, H * NH + 3>(op, tile);
  }
}
template <int KS, int J, int T, int FMT>
__device__ __forceinline__ void read_b(FragsB& b, const Operand<T, FMT, 4>& op, uint32_t tile) {
  b.f[J] = read_frag<KS, J>(op, tile);
  b.f[J + 1] = read_frag<KS, J + 1>(op, tile);
}
// acc (+)= a * b; FIRST: = (the matrix instruction takes a literal zero for its addend: no registers are cleared)
template <bool FIRST, bool HALF>
__device__ __forceinline__ void mfma1(f32x4& c, const u32x4& a, const u32x4& b) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (HALF) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), FIRST ? zero : c, 0, 0, 0);
  else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), FIRST ? zero : c, 0, 0, 0);
}
// row I of the sub-step's 16 x 16 products, every other one backwards: only one operand changes from one to the next
template <bool FIRST, bool HALF, int H, int I, int NH>
__device__ __forceinline__ void mfma_row(const FragsA<NH>& a, const FragsB& b, Acc<2 * NH>& acc) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = I & 1 ? 3 - q : q;
    mfma1<FIRST, HALF>(acc[H * NH + I][j], a.f[I], b.f[j]);
  }
}
template <bool FIRST, bool HALF, int H, int NH>
__device__ __forceinline__ void mfma_block(const FragsA<NH>& a, const FragsB& b, Acc<2 * NH>& acc) {
  mfma_row<FIRST, HALF, H, 0>(a, b, acc);
  mfma_row<FIRST, HALF, H, 1>(a, b, acc);
  if constexpr (NH == 4) {
    mfma_row<FIRST, HALF, H, 2>(a, b, acc);
    mfma_row<FIRST, HALF, H, 3>(a, b, acc);
  }
}
// the 16 (8) MFMAs of a sub-step with this wave's 8 load instructions of one unit interleaved (two after each of the
// first pairs: how they are spread over the sub-step makes no measurable difference).  The wave runs this
// sub-step at raised priority: it then wins the SIMD's issue slots from the other wave group's wave, its loads
// leave early in the K-step and have the longest time to land (query-side GEMM 6 % faster, logit kernel 1 %;
// raising the priority of every MFMA block instead is 1-4 % slower everywhere)
template <bool FIRST, bool HALF, int H, int T, int FMT, int NFRAG, int NH>
__device__ __forceinline__ void mfma_block_loads(const FragsA<NH>& a, const FragsB& b, Acc<2 * NH>& acc, const Operand<T, FMT, NFRAG>& op,
                                                 __amdgpu_buffer_rsrc_t from, char* lds) {
#define DISCO_LD(n) op.load(n, from, lds)
#define DISCO_MM(i, j) mfma1<FIRST, HALF>(acc[H * NH + i][j], a.f[i], b.f[j])
  __builtin_amdgcn_s_setprio(1);
  DISCO_MM(0, 0); DISCO_MM(0, 1); DISCO_LD(0); DISCO_LD(1);
  DISCO_MM(0, 2); DISCO_MM(0, 3); DISCO_LD(2); DISCO_LD(3);
  DISCO_MM(1, 3); DISCO_MM(1, 2); DISCO_LD(4); DISCO_LD(5);
  DISCO_MM(1, 1); DISCO_MM(1, 0); DISCO_LD(6); DISCO_LD(7);
  if constexpr (NH == 4) {
    mfma_row<FIRST, HALF, H, 2>(a, b, acc);
    mfma_row<FIRST, HALF, H, 3>(a, b, acc);
  }
  __builtin_amdgcn_s_setprio(0);
#undef DISCO_LD
#undef DISCO_MM
}

__device__ __forceinline__ int ring_next(int u, int step) { u += step; return u >= NUNITS ? u - NUNITS : u; }

// The K loop of one wave group.  GROUP 0 (the lower half of the waves) loads the A units, GROUP 1 the B units.
//
// Ring of five units; the operand tiles are laid into it in the order A0 B0 A1 B1 A2 B2 ..., item n in
// unit n mod 5.  K-step kt computes from A(kt), B(kt) in four sub-steps, the upper and the lower half of the wave's A
// rows against its B rows over 32 of the reduction, then over the other 32 (so a B fragment serves two sub-steps and two
// sets of 32 registers hold the fragments in use and the ones under way), each fetching the next
// sub-step's fragments while its MFMAs run:
//   sub-step 0;
//   sub-step 1: group 0 issues the loads of A(kt+2) into the unit that held B(kt-1);
//   sub-step 2, then: wait for this wave's loads of K-step kt+1 (group 0 may leave the 8 loads of A(kt+2)
//       in flight, group 1 has nothing younger), wait for its own LDS reads, barrier: K-step kt+1 is complete
//       in LDS and nobody reads the units of K-step kt any more (the last fragments are in registers);
//   sub-step 3: group 1 issues the loads of B(kt+2) into the unit that held A(kt); the first fragments of
//       K-step kt+1 are fetched.
// So an A load has six sub-steps to land and a B load four.  The last two K-steps are a loop of their own that loads nothing
// (loading the last K-step again instead, for one loop, made a tile of 8 K-steps fetch 10: 1 % of a call at d = 512, 3 % at 128).
// READS_FIRST: issue a sub-step's LDS reads ahead of its MFMAs (otherwise the compiler places them).
//
// PS: the operands may be kept as several 16-bit planes (a value is the sum of its planes, to their last bit), `plane_a` / `plane_b` elements
// apart, and PS lists the plane products that make up one K-step's worth of the reduction: the loop then runs PS::N
// times the K-steps: the products of one 64-deep piece one after the other, so that each plane's piece comes from L2 when it
// is read again, or (PS::SWEEPS) one product over the whole reduction after the other, so that the smallest products are
// added up while the sum is small and only the last sweep rounds at the size of the result.
template <int FMT>
__device__ __forceinline__ int64_t kstep_elems(int64_t ld) {
  return FMT == FMT_K ? BK : FMT == FMT_KA ? 4096 : FMT == FMT_R ? (int64_t)BK * ld : ld;
}

// WRITE_FIRST: the first K-step is peeled off the loop and writes the accumulators (acc = product, acc need not be
// initialised); else every K-step adds to them (acc += product).  Peeling gains 2-5 % on the gradient GEMMs; in the
// logit kernel it costs the epilogue registers it does not have.
template <int T, int FA, int FB, int GROUP, bool READS_FIRST, bool WRITE_FIRST, class PS, class BD, class SH>
__device__ __forceinline__ void kloop(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ Bp, int64_t ldb,
                                      int ktiles, char* smem, Acc<Cfg<T>::NFA>& acc, int nvalid_b, int64_t plane_a, int64_t plane_b, const BD& bounds, const SH& shifts) {
  static_assert(!BD::ON || PS::N == 1);
  static_assert(!SH::ON || (PS::HALF && FB == FMT_R));
  constexpr int NFA = Cfg<T>::NFA, NH = NFA / 2, WN = Cfg<T>::WN, UNIT_BYTES = Cfg<T>::UNIT_BYTES;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t stepA = kstep_elems<FA>(lda);
  const int64_t stepB = kstep_elems<FB>(ldb);
  const int last = ktiles - 1;
  // operand tiles of step kt: with several planes, product q of a 64-deep piece
  const int pieces = ktiles / PS::N;
  const uint32_t inv = 0xffffffffu / (uint32_t)pieces + 1u;      // (kt pieces < 2^32, which who makes the plans sees to: the high half of kt inv is the quotient)
  struct Step { int piece, q; };
  auto step_of = [&](int kt) {
    const int x = !PS::SWEEPS ? kt / PS::N : pieces == 1 ? kt : (int)__umulhi((uint32_t)kt, inv), y = kt - x * (PS::SWEEPS ? pieces : PS::N);
    return PS::SWEEPS ? Step{y, x} : Step{x, y};
  };
  auto tile_a = [&](int kt) {
    if constexpr (PS::N == 1) return A + kt * stepA;
    else { const auto [piece, q] = step_of(kt); return A + piece * stepA + (PS::A >> (2 * q) & 3) * plane_a; }
  };
  auto tile_b = [&](int kt) {
    if constexpr (PS::N == 1) return Bp + kt * stepB;
    else { const auto [piece, q] = step_of(kt); return Bp + piece * stepB + (PS::B >> (2 * q) & 3) * plane_b; }
  };
  auto from_a = [&](int kt) {
    if constexpr (BD::ON) return buffer_at(tile_a(kt), bytes_left<T, FA>(bounds.rows_a, 0u, lda, kt));
    else return buffer_at(tile_a(kt));
  };
  auto from_b = [&](int kt) {
    if constexpr (BD::ON) return buffer_at(tile_b(kt), bytes_left<T, FB>(bounds.rows_b, bounds.col_b, ldb, kt));
    else return buffer_at(tile_b(kt));
  };
  Operand<T, FA, NFA> oa;
  Operand<T, FB, 4> ob;
  oa.init(lda, wave % WN, lane, (wave / WN) * Cfg<T>::WTM);
  ob.init(ldb, wave % WN, lane, (wave % WN) * 64, nvalid_b);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;   // LDS byte address
  const int k1 = last < 1 ? last : 1;
  if (GROUP == 0) {
    oa.load_all(from_a(0), smem);
    oa.load_all(from_a(k1), smem + 2 * UNIT_BYTES);
  } else {
    ob.load_all(from_b(0), smem + UNIT_BYTES);
    ob.load_all(from_b(k1), smem + 3 * UNIT_BYTES);
  }
  wait_vmcnt<NLD>();
  if constexpr (SH::ON && GROUP == 1) shift_rows<T>(fetch_exponents<T>(shifts, step_of(0).piece, wave % WN), shifts.least, smem + UNIT_BYTES, wave % WN, lane);
  lds_barrier();
  FragsA<NH> a0, a1;
  FragsB b0, b1;
  read_a<0, 0>(a0, oa, smem_addr);
  read_b<0, 0>(b0, ob, smem_addr + UNIT_BYTES);
  read_b<0, 2>(b0, ob, smem_addr + UNIT_BYTES);
  wait_frags(a0, b0);

  auto next_exponents = [&](int kt) {               // of the K-step after kt
    if constexpr (SH::ON && GROUP == 1) return fetch_exponents<T>(shifts, step_of(kt < last ? kt + 1 : last).piece, wave % WN);
    else return 0;
  };
  int rA = 0;                                       // unit of A(kt); B(kt) is the next unit of the ring
  // One K-step (FIRST: its first products write the accumulators instead of adding to them; LOADS: it asks for K-step kt + 2, or,
  // in a reduction of one or two, which the first K-step of WRITE_FIRST may be, for the last again, into units nobody reads).  On entry a0 and b0 hold the first
  // half's fragments of the A side's upper rows and of the B side.
#define DISCO_KSTEP(FIRST, LOADS)                                                                                             \
  {                                                                                                                        \
    const int rB = ring_next(rA, 1), nA = ring_next(rA, 2), nB = ring_next(rA, 3), lA = ring_next(rA, 4);                  \
    const uint32_t ta = smem_addr + (uint32_t)(rA * UNIT_BYTES), tb = smem_addr + (uint32_t)(rB * UNIT_BYTES);             \
    const uint32_t tna = smem_addr + (uint32_t)(nA * UNIT_BYTES), tnb = smem_addr + (uint32_t)(nB * UNIT_BYTES);           \
    const int kload = kt + 2 < ktiles ? kt + 2 : last;                                                                     \
    const auto exponents = next_exponents(kt);                                                                             \
    /* sub-step 0 */                                                                                                       \
    read_a<0, 1>(a1, oa, ta);                                                                                              \
    read_b<1, 0>(b1, ob, tb);                                                                                              \
    if (READS_FIRST) __builtin_amdgcn_sched_barrier(0);                                                                    \
    mfma_block<FIRST, PS::HALF, 0>(a0, b0, acc);                                                                                     \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    wait_frags(a1, b0);                                                                                                    \
    /* sub-step 1 */                                                                                                       \
    read_a<1, 0>(a0, oa, ta);                                                                                              \
    read_b<1, 2>(b1, ob, tb);                                                                                              \
    if (READS_FIRST) __builtin_amdgcn_sched_barrier(0);                                                                    \
    if (GROUP == 0 && LOADS) mfma_block_loads<FIRST, PS::HALF, 1>(a1, b0, acc, oa, from_a(kload), smem + lA * UNIT_BYTES);                    \
    else mfma_block<FIRST, PS::HALF, 1>(a1, b0, acc);                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    wait_frags(a0, b1);                                                                                                    \
    /* sub-step 2 */                                                                                                       \
    read_a<1, 1>(a1, oa, ta);                                                                                              \
    if (READS_FIRST) __builtin_amdgcn_sched_barrier(0);                                                                    \
    mfma_block<false, PS::HALF, 0>(a0, b1, acc);                                                                                     \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    if (GROUP == 0 && LOADS) wait_vmcnt<NLD>(); else wait_vmcnt<0>();                                                               \
    wait_frags(a1, b1);                                                                                                    \
    if constexpr (SH::ON && GROUP == 1) {                                                                                  \
      shift_rows<T>(exponents, shifts.least, smem + nB * UNIT_BYTES, wave % WN, lane);                                     \
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                                                   \
    }                                                                                                                      \
    asm volatile("s_barrier" ::: "memory");                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    /* sub-step 3 */                                                                                                       \
    read_a<0, 0>(a0, oa, tna);                                                                                             \
    read_b<0, 0>(b0, ob, tnb);                                                                                             \
    read_b<0, 2>(b0, ob, tnb);                                                                                             \
    if (READS_FIRST) __builtin_amdgcn_sched_barrier(0);                                                                    \
    if (GROUP == 1 && LOADS) mfma_block_loads<false, PS::HALF, 1>(a1, b1, acc, ob, from_b(kload), smem + rA * UNIT_BYTES);                    \
    else mfma_block<false, PS::HALF, 1>(a1, b1, acc);                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    wait_frags(a0, b0);                                                                                                    \
    __builtin_amdgcn_sched_barrier(0);                                                                                     \
    rA = nA;                                                                                                               \
  }
  if constexpr (WRITE_FIRST) {
    // (the K-step as a generic lambda instantiated twice: this form, not only the peeling, is what the compiler
    // schedules 2-5 % better in the gradient GEMMs)
    auto kstep = [&](int kt, auto first, auto loads) { DISCO_KSTEP(decltype(first)::value, decltype(loads)::value) };
    kstep(0, std::true_type{}, std::true_type{});
    int kt = 1;
    for (; kt + 2 < ktiles; ++kt) kstep(kt, std::false_type{}, std::true_type{});
    for (; kt < ktiles; ++kt) kstep(kt, std::false_type{}, std::false_type{});
  } else {
    int kt = 0;
    for (; kt + 2 < ktiles; ++kt) DISCO_KSTEP(false, true)
    for (; kt < ktiles; ++kt) DISCO_KSTEP(false, false)
  }
#undef DISCO_KSTEP
  wait_vmcnt<0>();
  lds_barrier();
}

// acc[bm][bn] (+)= A_tile(T x K) * B_tile(T x K)^T for this wave's T/2 x 64 piece (WRITE_FIRST: =, see kloop).
//   FA / FB : tile format of the A / B operand (FMT_K: element (r,k) at base[r*ld + k]; FMT_R: at base[k*ld + r];
//             FMT_KA / FMT_RA: the same for storage in 16-byte atoms, see the top of this file).
//   A, Bp   : element (row 0, k 0) of the workgroup's operand tiles; ktiles = PS::N K / 64 >= 1.
//   smem    : Cfg<T>::SMEM_BYTES of LDS, 16-byte aligned; on return no load is in flight and every wave has passed
//             a barrier, so the caller may reuse it at once.
//   nvalid_b: rows of the B tile that exist in memory (multiple of 8, <= T); the output columns from
//             nvalid_b on are then meaningless and must not be stored.
//   bounds  : see Whole and Bounded.
//   shifts  : see Unshifted and RowShifts.
template <int T, int FA, int FB, bool READS_FIRST, bool WRITE_FIRST = false, class PS = Planes<1, 1>, class BD = Whole, class SH = Unshifted>
__device__ __forceinline__ void mainloop(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ Bp,
                                         int64_t ldb, int ktiles, char* smem, Acc<Cfg<T>::NFA>& acc, int nvalid_b = T,
                                         int64_t plane_a = 0, int64_t plane_b = 0, const BD& bounds = BD{}, const SH& shifts = SH{}) {
  if (threadIdx.x < Cfg<T>::NTHREADS / 2) kloop<T, FA, FB, 0, READS_FIRST, WRITE_FIRST, PS, BD, SH>(A, lda, Bp, ldb, ktiles, smem, acc, nvalid_b, plane_a, plane_b, bounds, shifts);
  else kloop<T, FA, FB, 1, READS_FIRST, WRITE_FIRST, PS, BD, SH>(A, lda, Bp, ldb, ktiles, smem, acc, nvalid_b, plane_a, plane_b, bounds, shifts);
}

// Writes a workgroup's T x T fp32 accumulator tile to row-major global memory through LDS, so that
// every global store is a full 1 KiB (T = 128: 512-byte) row segment (the accumulator layout would give 4-byte elements
// per lane).  Passes of 128 rows; LDS rows padded by 16 bytes so that the four rows of a wave's 4-byte
// write land on different banks.  out points at the tile's first element; value = scale * acc (+ old);
// only the first ncols columns (a multiple of 4) of the first nrows rows are touched.
template <int T>
constexpr int OUT_ROW_BYTES = T * 4 + 16;
template <int T>
constexpr int OUT_SMEM_BYTES = 128 * OUT_ROW_BYTES<T>;       // 132 KiB (T = 128: 68 KiB)

template <int T, bool ACCUMULATE, bool ROWMASK>
__device__ __forceinline__ void store_tile_f32_rows(Acc<Cfg<T>::NFA>& acc, char* smem, float* out, int64_t ld, float scale, int ncols, int nrows) {
  constexpr int WN = Cfg<T>::WN, NFA = Cfg<T>::NFA, RB = OUT_ROW_BYTES<T>;
  constexpr int CPR = T / 4, RSTEP = Cfg<T>::NTHREADS / CPR;      // 16-byte pieces per row, rows the workgroup stores at a time (8)
  constexpr int PASSES = T / 128;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int chunk = t % CPR, r0 = t / CPR;
  const bool live = chunk * 4 < ncols;             // this thread's four columns exist (ncols is a multiple of 4)
#pragma unroll
  for (int h = 0; h < PASSES; ++h) {
    // when accumulating, the old values are requested eight rows at a time, the first eight before the
    // staging so that their latency is paid under the LDS traffic
    f32x4 old[8];
    if (ACCUMULATE && live) {
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (!ROWMASK || h * 128 + r * RSTEP + r0 < nrows) old[r] = *reinterpret_cast<const f32x4*>(out + (int64_t)(h * 128 + r * RSTEP + r0) * ld + chunk * 4);
    }
    lds_barrier();
    if (PASSES == 1 || wm == h) {
      const int rbase = PASSES == 1 ? wm * Cfg<T>::WTM : 0;
      char* dst = smem + (rbase + (lane >> 4) * 4) * RB + (wn * 64 + (lane & 15)) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NFA; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) *reinterpret_cast<float*>(dst + (i * 16 + r) * RB + j * 64) = scale * acc[i][j][r];
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f32x4 v[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = *reinterpret_cast<const f32x4*>(smem + ((q * 8 + r) * RSTEP + r0) * RB + chunk * 16);
      if (ACCUMULATE && q == 1 && live) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          if (!ROWMASK || h * 128 + (8 + r) * RSTEP + r0 < nrows) old[r] = *reinterpret_cast<const f32x4*>(out + (int64_t)(h * 128 + (8 + r) * RSTEP + r0) * ld + chunk * 4);
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool there = live && (!ROWMASK || h * 128 + (q * 8 + r) * RSTEP + r0 < nrows);
        float* g = out + (int64_t)(h * 128 + (q * 8 + r) * RSTEP + r0) * ld + chunk * 4;
        if (ACCUMULATE && there) v[r] += old[r];
        if (there) *reinterpret_cast<f32x4*>(g) = v[r];
      }
    }
  }
}

// (a tile whose rows all exist takes the instance without the per-row tests)
template <int T, bool ACCUMULATE>
__device__ __forceinline__ void store_tile_f32(Acc<Cfg<T>::NFA>& acc, char* smem, float* out, int64_t ld, float scale, int ncols = T,
                                               int nrows = T) {
  if (nrows >= T) store_tile_f32_rows<T, ACCUMULATE, false>(acc, smem, out, ld, scale, ncols, nrows);
  else store_tile_f32_rows<T, ACCUMULATE, true>(acc, smem, out, ld, scale, ncols, nrows);
}

// Workgroup id -> tile, keeping the workgroups that share an XCD's L2 on neighbouring tiles.
// Workgroups are dealt round-robin to the 8 XCDs; XCD x takes the x-th contiguous eighth of the
// (padded) tile list.  Returns false for padding.
__device__ __forceinline__ bool xcd_linear(int w, int total, int& lin) {
  const int chunk = (total + 7) / 8;
  lin = (w & 7) * chunk + (w >> 3);
  return (w >> 3) < chunk && lin < total;
}

// Tile (it, jt) at position lin of the walk over super-blocks of sbi query tiles x sbj key tiles: bands of sbj key
// tiles one after the other, inside a band the super-blocks along the query tiles, inside a super-block the query
// tile runs fastest.  The last super-block of either direction may be partial.
__device__ __forceinline__ void superblock_tile(int lin, int nI, int nJ, int sbi, int sbj, int& it, int& jt) {
  const int band = sbj * nI;
  const int jb = lin / band, r = lin - jb * band;
  const int hj = nJ - jb * sbj < sbj ? nJ - jb * sbj : sbj;
  const int ib = r / (sbi * hj), r2 = r - ib * sbi * hj;
  const int wi = nI - ib * sbi < sbi ? nI - ib * sbi : sbi;
  it = ib * sbi + r2 % wi;
  jt = jb * sbj + r2 / wi;
}

// Time estimates in microseconds that the plans compare, for a chip of 256 compute units.  What they rest on (measured):
// a 64-deep K-step of a workgroup takes 1.15 (T = 256) or 0.57 (T = 128) where few workgroups run and 1.7 or 1.03 where
// every compute unit holds one (two), and prologue and store of a gradient tile another 8 or 3 (logit tiles 5.5 or 2.5).
// The figures carry b = 64 .. 8192 rows of 256 .. 196608 keys to within about 15 % of the tile kernels' time; a call takes about 21 us more in
// launches and small kernels, and the symmetric path its combining pass (3810 us against an estimate of 3009 at B = 32768, d = 512).  (They are of the loop on 32x32x16 products; on
// 16x16x32 ones both tile sizes take 8 % less, which leaves the choice between the sizes as it is: forcing each of the four pairs of tile
// sizes on 12 shapes beat the chosen plan by 4 % at most.  Against other kernels that factor does not cancel: those comparisons, of the
// small kernels with the tile paths and with the split kernels, carry allowances measured on the present kernels.)
constexpr double CHIP_CUS = 256.0;
constexpr double BYTES_PER_US = 4.5e6;

inline double step_us(int T, double wgs) {
  const double slots = T == 256 ? CHIP_CUS : 2 * CHIP_CUS, few = T == 256 ? 1.15 : 0.57, full = T == 256 ? 1.7 : 1.03;
  const double f = (wgs - slots / 4) / (slots * 3 / 4);
  return few + (full - few) * (f < 0 ? 0 : f > 1 ? 1 : f);
}

}  // namespace tile
}  // namespace disco

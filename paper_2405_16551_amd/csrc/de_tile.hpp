// de_tile.hpp -- device code shared by the per-problem and the batched
// generation kernels: vector helpers, the per-run statistics update and the
// rotated-objective tile (build trials into LDS, Z = Y R^T on MFMA with the
// objective fused, select and write).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "de_device.hpp"
#include "de_internal.h"

namespace de {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr unsigned long long kNoHit = ~0ull;

__device__ __forceinline__ float4 ld4(const float* p) {
  return *reinterpret_cast<const float4*>(p);
}
__device__ __forceinline__ void st4(float* p, float4 v) {
  *reinterpret_cast<float4*>(p) = v;
}
__device__ __forceinline__ float get(const float4& v, int b) {
  return b == 0 ? v.x : b == 1 ? v.y : b == 2 ? v.z : v.w;
}
__device__ __forceinline__ void set(float4& v, int b, float s) {
  if (b == 0) v.x = s; else if (b == 1) v.y = s; else if (b == 2) v.z = s;
  else v.w = s;
}

// Statistics after an accepted trial with value f of individual i in run r,
// which produced generation gen+1.
__device__ __forceinline__ void record_accept_at(const GenArgs& a, int run,
                                                 int i, float f,
                                                 uint32_t gen) {
  atomicAdd(&a.accepted[run], 1ull);
  atomicMin(&a.best_key[run], fit_key(f, i));
  if (f <= a.target) {
    const unsigned long long old =
        atomicMin(&a.hit_gen[run], (unsigned long long)gen + 1ull);
    if (old == kNoHit) atomicAdd(a.done, 1u);
  }
}

__device__ __forceinline__ void record_accept(const GenArgs& a, int run, int i,
                                              float f) {
  record_accept_at(a, run, i, f, a.gen);
}

// ---------------------------------------------------------------------------
// Rotated objective.  Tile of BM trial rows per workgroup of NT threads.
//   phase 1: donors of every row, then per row all target/donor loads in
//            flight before the crossover draws; trial rows -> LDS A tile as
//            y = u - o in the GEMM precision, crossover decisions -> bit
//            planes; padding rows and columns are zero.
//   phase 2: Z = Y R^T in 32x32 MFMA blocks, wave tile BM rows x one
//            32-column block per pass, R fragments prefetched from L2
//            (BF16: eight K-steps ahead); the
//            objective z^2 + sin^2(3z) is summed per row in registers.
//   phase 3: row totals -> selection -> next generation rows (a rejected row
//            is rewritten only if the other buffer holds a stale copy),
//            statistics.
// Operand precision of the rotation product: LDS element type and the parts
// an operand is held in.
struct PrecBF16 {
  using T = __bf16;
  static constexpr int kPad = 8;  // LDS row padding, elements
  static constexpr int kParts = 1;
};
// FP32 operands on the FP32 matrix instruction (fewer than kX3MinD coordinates).
struct PrecF32 {
  using T = float;
  static constexpr int kPad = 4;
  static constexpr int kParts = 1;
};
// FP32 operands on the BF16 matrix instruction: y = yh + ym + yl and R = Rh +
// Rm + Rl, three BF16 parts of eight significant bits each, which hold all 24
// bits of an FP32 value from 2^-102 up (the smallest part of a smaller one
// falls below BF16's least normal) to the largest (the splitting of Henry,
// Tang & Heinecke, "Leveraging the bfloat16 artificial intelligence datatype
// for higher-precision computations", ARITH 2019).  Per K-step of 16
// coordinates one MFMA forms yh Rh and a chain of seven the smaller products,
// both from zero; their sum is then added to z in FP32.
//   - Why: an FP32 MFMA runs at 1/16 of the BF16 rate and on the vector FMA
//     units (measured: FP32 MFMA next to FMAs of another wave takes the sum
//     of both times, half-precision MFMA the larger): 512 clocks a block and
//     K-step there, 256 here.  16 x 1024 x 1000: 303 us per generation there,
//     244 here, of which the eight products take 168 (1.6 PFLOP/s).
//   - Accuracy: of the nine products only yl Rl (2^-32 of a term) is left out,
//     products of parts are exact, and z is rounded twice per K-step instead
//     of 16 times.  The chain is apart because a BF16 MFMA does not round its
//     sum to nearest: with yh Rh in it a coordinate alone in its row would be
//     off by up to 1.1 half-ulps, where it is the rounded product so, as a
//     fused multiply-add's.  Error of f against 64 bits, root mean square in
//     2^-24, FP32 MFMA / here: dense R 0.95 / 0.81 (32 coordinates), 0.91 /
//     0.79 (100), 1.04 / 0.92 (256), 1.50 / 1.22 (700), 1.42 / 1.14 (1000);
//     diagonal R over three decades 0.89 / 0.89; permutations 0.42 / 0.42.
//     Six products would be faster (215 us) and worse for sparse R (0.94 ->
//     0.97), two half-precision parts (three products, 123 us) two bits short.
// Problems of kX3MinD coordinates and more; below, the FP32 instruction's
// chain is as short.
struct PrecX3 {
  using T = __bf16;
  static constexpr int kPad = 8;
  static constexpr int kParts = 3;
};
constexpr int kX3MinD = 32;
constexpr int kX3TallMinBlocks = 24;  // column blocks; beyond: 64-row tiles

// The three BF16 parts of N values, a pair at a time: the high part the upper
// half of the word (rounded it could overflow), the others rounded.
template <int N, class V>
__device__ __forceinline__ void x3_split(const float (&v)[N], V (&p)[3]) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float floatx2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int u = 0; u < N; u += 2) {
    float r0 = v[u], r1 = v[u + 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t w =
          q == 0 ? (__builtin_bit_cast(uint32_t, r0) >> 16) |
                       (__builtin_bit_cast(uint32_t, r1) & 0xFFFF0000u)
                 : __builtin_bit_cast(uint32_t, __builtin_convertvector(
                                                    (floatx2{r0, r1}), bf16x2));
      const bf16x2 h = __builtin_bit_cast(bf16x2, w);
      p[q][u] = h[0];
      p[q][u + 1] = h[1];
      r0 -= __builtin_bit_cast(
          float, q == 0 ? __builtin_bit_cast(uint32_t, r0) & 0xFFFF0000u
                        : w << 16);
      r1 -= __builtin_bit_cast(
          float, q == 0 ? __builtin_bit_cast(uint32_t, r1) & 0xFFFF0000u
                        : w & 0xFFFF0000u);
    }
  }
}

// Slots of the per-row objective sums (see rot_tile).
constexpr int kRotSlots = 16;

template <class P, int BM, bool JDE = false>
__host__ __device__ constexpr size_t rot_lds_bytes(int dpad) {
  const int tq = (dpad / 4 + 63) / 64;
  return (size_t)BM * (P::kParts * dpad + P::kPad) * sizeof(typename P::T)  // A
         + (size_t)BM * tq * 4 * sizeof(unsigned long long)     // planes
         + (size_t)BM * 4 * sizeof(int)                         // donors
         + (size_t)kRotSlots * BM * sizeof(float)               // slot sums
         + (JDE ? (size_t)BM * sizeof(Control) : 0);            // F', CR'
}

// Coordinates j0 .. j0 + 3 of an LDS row.  BF16: natural order.  Three parts:
// each group of 8 coordinates as its 8 high, 8 middle and 8 low parts.  FP32:
// within each group of 8, k = 2s + h is stored at 4h + s so that one lane's
// four K-steps of the 32x32x2 MFMA are one 16-byte read.
template <class P>
__device__ __forceinline__ void put_quad(typename P::T* arow, int j0,
                                         float4 y) {
  if constexpr (P::kParts == 3) {
    const float v[4] = {y.x, y.y, y.z, y.w};
    bf16x4 p[3];
    x3_split(v, p);
    bf16x4* d = reinterpret_cast<bf16x4*>(arow + 3 * (j0 & ~7) + (j0 & 7));
    d[0] = p[0];
    d[2] = p[1];
    d[4] = p[2];
  } else if constexpr (sizeof(typename P::T) == 2) {
    bf16x4 yb;
    yb[0] = (__bf16)y.x;
    yb[1] = (__bf16)y.y;
    yb[2] = (__bf16)y.z;
    yb[3] = (__bf16)y.w;
    *reinterpret_cast<bf16x4*>(arow + j0) = yb;
  } else {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int k = j0 + b;
      arow[(k & ~7) + (k & 1) * 4 + ((k & 7) >> 1)] = get(y, b);
    }
  }
}

// One coordinate of the rotated oscillating objective: z^2 + sin^2(3z).
// FP32 product: sin^2 from the reduction and series of sin_squared.
// BF16 product (z already carries BF16 operand rounding, relative error
// ~2^-8): the hardware sine, which takes its argument in turns; 3z / (2 pi)
// is reduced to [-1/2, 1/2] turns first (exact), the remaining error is the
// FP32 rounding of 3z / (2 pi), about 2^-24 |3z| radians.
template <bool kFastSin>
__device__ __forceinline__ float osc_term(float z) {
  if constexpr (kFastSin) {
    constexpr float kTurnsPer3z = 0x1.e8ec8ap-2f;  // 3 / (2 pi)
    const float turns = z * kTurnsPer3z;
    const float s = __builtin_amdgcn_sinf(turns - rintf(turns));
    return fmaf(z, z, s * s);
  } else {
    return fmaf(z, z, sin_squared(3.0f * z));
  }
}

template <bool kFastSin>
__device__ __forceinline__ void osc_accumulate(floatx16& part,
                                               const floatx16& c) {
#pragma unroll
  for (int r = 0; r < 16; ++r) part[r] += osc_term<kFastSin>(c[r]);
}

// Rows per producer step of BF16 tiles (128 registers per lane).
constexpr int kBf16Rows = 4;
// Threads of the BF16 rotated tile.  Each wave owns one column block per
// pass and four producer rows per step, within 128 registers, so four
// waves fit per SIMD.  The tile has 16 waves (measured faster at D = 1000
// than 8 waves with twice the registers each), or 8 when two tiles fit in
// a CU's LDS (padded width up to 512) and there are more tiles than CUs:
// then each CU holds two and one tile's loads overlap the other's MFMAs.
// The result does not depend on the choice (row sums add column blocks in
// a fixed order).
constexpr int kRotBf16Threads = 1024;
constexpr int kRotBf16ThreadsNarrow = 512;
constexpr int kRotBf16NarrowMaxDpad = 512;
// While tiles of half the height still find a CU each, BF16 tiles have 32 rows:
// the tile is a chain of round trips and of a wave's rows, and half the rows
// (two a wave instead of four) make it shorter; R is then streamed by twice the
// CUs, which would be idle otherwise.  Per generation, 64 / 32 rows: 1 x 250 x
// 100 6.1 / 5.0 us, 30 x 256 x 100 6.4 / 5.1, 16 x 500 x 333 16.6 / 11.9,
// 1 x 1024 x 1000 40.5 / 32.1, 8 x 1024 x 1000 (every CU) 41.4 / 36.5.  With more
// tiles than CUs the 64-row tile, which streams R once per 64 rows.  Rows' sums
// are formed alike, so the result does not depend on it.
__host__ __device__ constexpr bool rot_few_tiles(long long tiles32, int cus) {
  return tiles32 <= cus;
}
__host__ __device__ constexpr bool rot_bf16_narrow(int dpad, long long tiles,
                                                   int cus) {
  return dpad <= kRotBf16NarrowMaxDpad && tiles > cus;
}

// Scheduling pattern for one K-step: per row block one MFMA and its next A
// read (LDS), then the step's R load (L2), so the matrix unit keeps busy
// while the reads go out instead of waiting behind one burst.
template <int MB>
__device__ __forceinline__ void interleave_step() {
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
  __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
  if constexpr (MB == 2) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // VMEM read
  __builtin_amdgcn_sched_barrier(0);
}

// Two consecutive FP32 four-step groups (k8, k8 + 1) of one column block
// into two accumulators, interleaved.
__device__ __forceinline__ void f32_step2(const float* ar, int k8, float4 b0,
                                          float4 b1, floatx16& ce,
                                          floatx16& co) {
  const float4 a0 = *reinterpret_cast<const float4*>(ar + k8 * 8);
  const float4 a1 = *reinterpret_cast<const float4*>(ar + (k8 + 1) * 8);
  ce = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, b0.x, ce, 0, 0, 0);
  co = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, b1.x, co, 0, 0, 0);
  ce = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, b0.y, ce, 0, 0, 0);
  co = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, b1.y, co, 0, 0, 0);
  ce = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, b0.z, ce, 0, 0, 0);
  co = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, b1.z, co, 0, 0, 0);
  ce = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, b0.w, ce, 0, 0, 0);
  co = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, b1.w, co, 0, 0, 0);
}

// Widest padded row of the paired-row form: 32 quads, so that one row's
// quads fill half a wave and its crossover bits are one 32-bit half of a
// ballot.  Launchers refuse PAIR beyond it.
constexpr int kPairMaxDpad = 128;

// What the phases of a tile share about its rows.
struct RotRows {
  const float* base;             // the run's population (EVAL: the rows)
  int* donors;                   // LDS: r1, r2, r3, j_rand per row
  Control* ctl;                  // LDS, jDE: F', CR' per row
  unsigned long long* planes;    // LDS: crossover lane masks [row][chunk][4]
  uint32_t rng_run;
  int row0, nvalid, stride, tq;
};

// Chunk t (256 coordinates) of the wave's rows rl = wave + kWaves * k, RB
// rows at a time, into the A tile, whose column 0 is coordinate 0 of At0.
template <class P, int RB, int kWaves, bool EVAL, bool JDE>
__device__ __forceinline__ void build_chunk(const GenArgs& a, const RotRows& c,
                                            int t, typename P::T* At0) {
  using T = typename P::T;
  const int wave = (int)threadIdx.x / 64, lane = (int)threadIdx.x % 64;
  const int nrow_w =
      wave < c.nvalid ? (c.nvalid - 1 - wave) / kWaves + 1 : 0;
  const int dlast = ((a.D + 3) / 4 - 1) * 4;
  const int q = lane + 64 * t, j0 = 4 * q, jl = min(j0, dlast);
  const float4 ov = ld4(a.o + jl);
  // a chunk with the row's end: its coordinates past D are zeroed
  const bool whole = 256 * (t + 1) <= a.D;
  XoverCol xc{0, 0, 0, 0};
  if (!EVAL)
    xc = xover_col(c.rng_run, a.gen, (uint32_t)q, a.key_lo, a.key_hi);
  for (int k = 0; k < nrow_w; k += RB) {
    float4 xv[RB], v1[RB], v2[RB], v3[RB];
#pragma unroll
    for (int h = 0; h < RB; ++h) {
      // row and donor indices are wave-uniform: scalar row pointers
      const int rl = __builtin_amdgcn_readfirstlane(
          wave + kWaves * min(k + h, nrow_w - 1));
      xv[h] = ld4(c.base + (size_t)(c.row0 + rl) * a.ldx + jl);
      if (!EVAL) {
        v1[h] = ld4(c.base + (size_t)__builtin_amdgcn_readfirstlane(
                               c.donors[rl * 4 + 0]) * a.ldx + jl);
        v2[h] = ld4(c.base + (size_t)__builtin_amdgcn_readfirstlane(
                               c.donors[rl * 4 + 1]) * a.ldx + jl);
        v3[h] = ld4(c.base + (size_t)__builtin_amdgcn_readfirstlane(
                               c.donors[rl * 4 + 2]) * a.ldx + jl);
      }
    }
    // every gather of the step is issued before any of it is used:
    // keeps the compiler from sinking a row's loads into the guarded
    // code that consumes them
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < RB; ++h) {
      if (k + h >= nrow_w) break;
      const int rl =
          __builtin_amdgcn_readfirstlane(wave + kWaves * (k + h));
      T* arow = At0 + (size_t)rl * c.stride;
      float4 y;
      if constexpr (EVAL) {
#pragma unroll
        for (int b = 0; b < 4; ++b) set(y, b, get(xv[h], b) - get(ov, b));
      } else {
        const int jrand = c.donors[rl * 4 + 3];
        float Fr = a.F;
        uint32_t limit = xover_word_limit(a.cr_threshold);
        if constexpr (JDE) {
          Fr = c.ctl[rl].F;
          limit = xover_word_limit(cr_threshold_of(c.ctl[rl].CR));
        }
        const XoverRow xr = xover_row(a.gen, (uint32_t)(c.row0 + rl),
                                      a.key_lo, a.key_hi);
        const Words4 w = xover_words(xc, xr, a.key_lo, a.key_hi);
        unsigned long long m[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          // bitwise & and |: the tests are lane masks, no branch
          const bool tk = (j0 + b < a.D) &
                          ((j0 + b == jrand) | (w.w[b] <= limit));
          const float mv = mutant_coord(get(v1[h], b), get(v2[h], b),
                                        get(v3[h], b), Fr, a.lo, a.hi);
          m[b] = __ballot(tk);
          set(y, b, (tk ? mv : get(xv[h], b)) - get(ov, b));
        }
        // the chunk's crossover planes: the decisions' lane masks,
        // stored by lane 0 as two 16-byte writes
        if (lane == 0) {
          ulonglong2* pp = reinterpret_cast<ulonglong2*>(
              c.planes + ((size_t)rl * c.tq + t) * 4);
          pp[0] = make_ulonglong2(m[0], m[1]);
          pp[1] = make_ulonglong2(m[2], m[3]);
        }
      }
      if (!whole) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          set(y, b, j0 + b < a.D ? get(y, b) : 0.f);
      }
      if (j0 < a.dpad) put_quad<P>(arow, j0, y);
    }
  }
}

// The objective of two 32x32 blocks' values (kHi: hi is there) summed over
// the 32 columns: a reduce-scatter butterfly leaves lane l with the total of
// value l % 32 (0-15: lo's registers, 16-31: hi's).
template <int m>
__device__ __forceinline__ void scatter_step(float (&v)[16], int lane) {
  const bool upper = (lane & m) != 0;
#pragma unroll
  for (int k = 0; k < m; ++k) {
    const float send = upper ? v[k] : v[k + m];
    const float keep = upper ? v[k + m] : v[k];
    v[k] = keep + lane_xor<m>(send);
  }
}

template <bool kFastSin, bool kHi>
__device__ __forceinline__ float osc_rows(const floatx16& lo,
                                          const floatx16& hi, int lane) {
  float v[16];
  // first exchange: values 0-15 keep lo or hi, the other half goes over
  const bool upper = (lane & 16) != 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float a = osc_term<kFastSin>(lo[k]);
    const float b = kHi ? osc_term<kFastSin>(hi[k]) : 0.f;
    v[k] = (upper ? b : a) + lane_xor<16>(upper ? a : b);
  }
  scatter_step<8>(v, lane);
  scatter_step<4>(v, lane);
  scatter_step<2>(v, lane);
  scatter_step<1>(v, lane);
  return v[0];
}

// The wave's rows in the selection: lane r < count has row wave + kWaves r,
// with its target's value and stale flag, read before the product so that
// the selection does not wait for them.
struct SelectRow {
  int rl;
  bool in;
  float fx;
  bool stale;
};

template <int kWaves, bool EVAL>
__device__ __forceinline__ SelectRow select_row(const GenArgs& a, int run,
                                                int row0, int nvalid) {
  const int wave = (int)threadIdx.x / 64, lane = (int)threadIdx.x % 64;
  SelectRow s;
  s.rl = wave + kWaves * lane;
  s.in = s.rl < nvalid;
  s.rl = s.in ? s.rl : wave;
  s.fx = 0.f;
  s.stale = false;
  if (!EVAL && s.in) {
    const size_t g = (size_t)run * a.NP + row0 + s.rl;
    s.fx = a.fit_cur[g];
    s.stale = a.changed[g] != 0;
  }
  return s;
}

// Writes the rows of `need` (bit r: row wave + kWaves r) into the next
// generation: trials (rebuilt from the crossover masks and the donors) where
// bit r of `accept` is set, else the target.  R rows at a time, so that the
// rows' reads share one round trip (four 256-coordinate pieces in flight).
template <int R, int kWaves, bool JDE>
__device__ __forceinline__ void write_rows(const GenArgs& a, const RotRows& c,
                                           int run, uint32_t need,
                                           uint32_t accept) {
  constexpr int C = 4 / R;  // chunks of a row in flight
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int lane = (int)threadIdx.x % 64;
  const int dlast = ((a.D + 3) / 4 - 1) * 4;
  while (need) {
    int rl[R];
    const float *x0[R], *x1[R], *x2[R], *x3[R];  // scalar row pointers
    bool on[R], acc[R];
#pragma unroll
    for (int h = 0; h < R; ++h) {
      on[h] = need != 0;
      const int r = on[h] ? __builtin_ctz(need) : 0;
      acc[h] = on[h] && ((accept >> r) & 1u);
      rl[h] = wave + kWaves * r;
      need &= need - 1;
      const int* d = c.donors + rl[h] * 4;
      x0[h] = c.base + (size_t)(c.row0 + rl[h]) * a.ldx;
      x1[h] = c.base + (size_t)__builtin_amdgcn_readfirstlane(d[0]) * a.ldx;
      x2[h] = c.base + (size_t)__builtin_amdgcn_readfirstlane(d[1]) * a.ldx;
      x3[h] = c.base + (size_t)__builtin_amdgcn_readfirstlane(d[2]) * a.ldx;
    }
    for (int t0 = 0; t0 < c.tq; t0 += C) {
      float4 xv[4], v1[4], v2[4], v3[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int h = s / C, t = t0 + s % C;
        // (past the row's end its last piece, past the last row row 0)
        const int jl = min(4 * (lane + 64 * t), dlast);
        if (on[h]) xv[s] = ld4(x0[h] + jl);
        if (acc[h]) {
          v1[s] = ld4(x1[h] + jl);
          v2[s] = ld4(x2[h] + jl);
          v3[s] = ld4(x3[h] + jl);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int h = s / C, t = t0 + s % C;
        const int j0 = 4 * (lane + 64 * t);
        if (!on[h] || t >= c.tq) continue;
        float4 out = xv[s];
        if (acc[h]) {
          const float Fr = JDE ? c.ctl[rl[h]].F : a.F;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const unsigned long long m =
                c.planes[((size_t)rl[h] * c.tq + t) * 4 + b];
            const float mv = mutant_coord(get(v1[s], b), get(v2[s], b),
                                          get(v3[s], b), Fr, a.lo, a.hi);
            set(out, b, ((m >> lane) & 1ull) ? mv : get(xv[s], b));
          }
        }
        if (j0 < a.D)
          st4(a.pop_next +
                  ((size_t)run * a.NP + c.row0 + rl[h]) * a.ldx + j0,
              out);
      }
    }
  }
}

// Row totals (slots added in order), strict selection, the next generation's
// rows (a rejected row only if the other buffer holds a stale copy) and the
// statistics; EVAL: the values alone.  All of the wave's rows are decided at
// once, one per lane.
template <int BM, int kWaves, bool EVAL, bool JDE>
__device__ __forceinline__ void select_rows(const GenArgs& a, const RotRows& c,
                                            int run, const float* fpart,
                                            const SelectRow& s) {
  float f = 0.f;
#pragma unroll
  for (int sl = 0; sl < kRotSlots; ++sl) f += fpart[sl * BM + s.rl];
  const int i = c.row0 + s.rl;
  if constexpr (EVAL) {
    if (s.in) a.fit_next[i] = f;
  } else {
    const bool accept = s.in && f < s.fx;
    if (s.in) {
      const size_t g = (size_t)run * a.NP + i;
      a.fit_next[g] = accept ? f : s.fx;
      a.changed[g] = accept ? 1 : 0;
      if constexpr (JDE) {
        // the trial's F', CR' survive only with the trial
        a.jp_next[g] = accept ? make_float2(c.ctl[s.rl].F, c.ctl[s.rl].CR)
                              : a.jp_cur[g];
      }
    }
    const uint32_t acc = (uint32_t)__ballot(accept);
    const uint32_t need = acc | (uint32_t)__ballot(s.in && s.stale);
    if (c.tq == 1)
      write_rows<4, kWaves, JDE>(a, c, run, need, acc);
    else if (c.tq == 2)
      write_rows<2, kWaves, JDE>(a, c, run, need, acc);
    else
      write_rows<1, kWaves, JDE>(a, c, run, need, acc);
    if (accept) record_accept(a, run, i, f);
  }
}

// z += Y R^T over `steps` K-steps for NB column blocks of R and MB row blocks
// (three-part operands).  ar: the lane's first fragment of the A rows (row l %
// 32, coordinates 8 (l / 32) on), row32 elements to the next row block.  rb:
// the first block's fragments, FP32, [K-step][half][64 lanes] of four
// coordinates each, bstep float4s to the next block.  R stays FP32 in memory
// (four bytes an element to stream instead of six) and is split by the one
// wave of the tile that multiplies by it.
// A block's R registers are loaded for the next step once all of them are
// split, without a branch and in the loop's order, so that the loads in
// flight can be counted.  Only the first `mine` blocks (NB or NB - 1) are
// multiplied; the loads of a missing last one repeat the one
// before it.
// (pin: the compiler otherwise puts the parts off until after the loads and
// the sums until the end of the step, and moves or spills what they hold.)
template <class V>
__device__ __forceinline__ void pin(V& v) {
  asm volatile("" : "+v"(v));
}

template <int MB, int NB>
__device__ __forceinline__ void x3_product(floatx16 (&acc)[NB][MB],
                                           const __bf16* ar, int row32,
                                           const float4* rb, size_t bstep,
                                           int steps, int lane, int mine) {
  // scalar row addresses, the lane's part in one register
  const uint32_t lofs = (uint32_t)lane * 16u;
  auto frag = [&](const float4* p) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(p) +
                                            lofs);
  };
  const size_t last = (size_t)(mine - 1) * bstep;
  float4 r[NB][2];
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      r[n][p] = frag(rb + (n < mine ? n * bstep : last) + 64 * p);
      __builtin_amdgcn_sched_barrier(0);
    }
  for (int s = 0; s < steps; ++s) {
    bf16x8 x[MB][3];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        x[m][p] =
            *reinterpret_cast<const bf16x8*>(ar + m * row32 + 48 * s + 8 * p);
    const float4* rn = rb + (size_t)(s + 1 < steps ? s + 1 : s) * 128;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const float v[8] = {r[n][0].x, r[n][0].y, r[n][0].z, r[n][0].w,
                          r[n][1].x, r[n][1].y, r[n][1].z, r[n][1].w};
      bf16x8 b[3];
      x3_split(v, b);
#pragma unroll
      for (int p = 0; p < 3; ++p) pin(b[p]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < 2; ++p)
        r[n][p] = frag(rn + (n < mine ? n * bstep : last) + 64 * p);
      if (NB > 1 && n == NB - 1 && n >= mine) break;
      constexpr int kA[7] = {1, 2, 2, 0, 1, 1, 0};
      constexpr int kB[7] = {2, 1, 0, 2, 1, 0, 1};
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        floatx16 t = {};
#pragma unroll
        for (int q = 0; q < 7; ++q)
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][kA[q]], b[kB[q]], t,
                                                      0, 0, 0);
        const floatx16 h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            x[m][0], b[0], floatx16{}, 0, 0, 0);
        acc[n][m] += h + t;
        pin(acc[n][m]);
      }
    }
  }
}

// One tile: rows row0 .. row0 + nvalid - 1 of run `run` (EVAL: of the
// flattened row range).  Ends with every LDS access of the tile complete
// only for the calling thread: a caller that runs another tile in the same
// workgroup synchronises first.  PAIR (padded widths up to kPairMaxDpad
// only): the trials are built two rows per wave instruction.
template <class P, int BM, int NT, bool EVAL, bool JDE = false,
          bool PAIR = false>
__device__ __forceinline__ void rot_tile(const GenArgs& a, int run, int row0,
                                         int nvalid) {
  using T = typename P::T;
  constexpr int MB = BM / 32;
  constexpr int kRotThreads = NT;
  constexpr int kRotWaves = NT / 64;
  static_assert(P::kParts == 1 || PAIR, "three parts: rot_tile_x3");
  static_assert(MB == 1 || (MB == 2 && sizeof(T) == 2), "tile shape");
  extern __shared__ __align__(16) char smem[];
  const int dpad = a.dpad;
  const int stride = P::kParts * dpad + P::kPad;
  const int tq = (dpad / 4 + 63) / 64;
  T* At = reinterpret_cast<T*>(smem);
  unsigned long long* planes = reinterpret_cast<unsigned long long*>(
      smem + (size_t)BM * stride * sizeof(T));
  int* donors = reinterpret_cast<int*>(planes + (size_t)BM * tq * 4);
  float* fpart = reinterpret_cast<float*>(donors + BM * 4);
  // jDE: the F' and CR' of every row of the tile
  Control* ctl = reinterpret_cast<Control*>(fpart + kRotSlots * BM);

  const int wave = (int)threadIdx.x / 64, lane = (int)threadIdx.x % 64;
  const uint32_t rng_run = a.run_base + (uint32_t)run;
  const float* base = a.pop_cur + (EVAL ? 0 : (size_t)run * a.NP * a.ldx);

  // ---- phase 1: build the A tile
  if (!EVAL) {
    for (int rl = (int)threadIdx.x; rl < nvalid; rl += kRotThreads) {
      const Donors d = pick_donors(rng_run, a.gen, row0 + rl, a.NP, a.D,
                                   a.key_lo, a.key_hi);
      donors[rl * 4 + 0] = d.r1;
      donors[rl * 4 + 1] = d.r2;
      donors[rl * 4 + 2] = d.r3;
      donors[rl * 4 + 3] = d.jrand;
      if constexpr (JDE) {
        const float2 c = a.jp_cur[(size_t)run * a.NP + row0 + rl];
        ctl[rl] = jde_control(rng_run, a.gen, row0 + rl, a.key_lo, a.key_hi,
                              a.jF_lo, a.jF_span, a.jtau_F, a.jtau_CR,
                              Control{c.x, c.y});
      }
    }
    __syncthreads();
  }
  // rows past the tile's last are zero
  for (int rl = nvalid + (((wave - nvalid) % kRotWaves) + kRotWaves) %
                             kRotWaves;
       rl < BM; rl += kRotWaves) {
    T* arow = At + (size_t)rl * stride;
    for (int k = lane; k < P::kParts * dpad; k += 64) arow[k] = (T)0.0f;
  }
  // PAIR: each wave keeps its rows' targets and trials (lane 32 h + q: quad
  // q of the h-th row of a pair), their values and stale flags in registers
  // from the build to the selection, which then reads no memory: the tile
  // is a chain of memory round trips (64 x 256 x 100, FP32: 12.6 us per
  // generation with the rows read again for the selection, 1 run x 250 x 100
  // in BF16 7.4 us), so the chain's length is what counts.
  constexpr int RBP = PAIR ? BM / (2 * kRotWaves) : 1;  // pairs per wave
  static_assert(!PAIR || (BM % (2 * kRotWaves) == 0 && RBP >= 1), "pairs");
  float4 pu[RBP], px[RBP];
  float pf[RBP];
  bool pchg[RBP];
  const int hl = lane / 32, ql = lane % 32;
  if constexpr (PAIR) {
    // Padded widths up to 128 (at most 32 quads per row): lanes 32 h + q
    // build quad q of the h-th row of a pair of the wave's rows, so every
    // lane has a quad (one row per instruction would leave more than half
    // of them idle).  Same loads, draws, arithmetic and stores as below.
    static_assert(!EVAL, "paired form: generation step");
    const int nrow_w = wave < nvalid ? (nvalid - 1 - wave) / kRotWaves + 1 : 0;
    if (nrow_w > 0) {
      const int dlast = ((a.D + 3) / 4 - 1) * 4;
      const int j0 = 4 * ql, jl = min(j0, dlast);
      const float4 ov = ld4(a.o + jl);
      float4 v1[RBP], v2[RBP], v3[RBP];
#pragma unroll
      for (int p = 0; p < RBP; ++p) {
        const int rl = wave + kRotWaves * min(2 * p + hl, nrow_w - 1);
        px[p] = ld4(base + (size_t)(row0 + rl) * a.ldx + jl);
        v1[p] = ld4(base + (size_t)donors[rl * 4 + 0] * a.ldx + jl);
        v2[p] = ld4(base + (size_t)donors[rl * 4 + 1] * a.ldx + jl);
        v3[p] = ld4(base + (size_t)donors[rl * 4 + 2] * a.ldx + jl);
      }
#pragma unroll
      for (int p = 0; p < RBP; ++p) {
        const int rl = wave + kRotWaves * min(2 * p + hl, nrow_w - 1);
        const size_t g = (size_t)run * a.NP + row0 + rl;
        pf[p] = a.fit_cur[g];
        pchg[p] = a.changed[g] != 0;
      }
#pragma unroll
      for (int p = 0; p < RBP; ++p) {
        if (2 * p >= nrow_w) break;
        const bool live = 2 * p + hl < nrow_w;  // the second row may not exist
        const int rl = wave + kRotWaves * min(2 * p + hl, nrow_w - 1);
        const int i = row0 + rl;
        const int jrand = donors[rl * 4 + 3];
        float Fr = a.F;
        uint32_t crt = a.cr_threshold;
        if constexpr (JDE) {  // the row's own F', CR'
          const Control c = ctl[rl];
          Fr = c.F;
          crt = cr_threshold_of(c.CR);
        }
        const Words4 w = draw_block(kTagXover, rng_run, a.gen, (uint32_t)i,
                                    (uint32_t)ql, a.key_lo, a.key_hi);
        float4 y;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const bool tk = (j0 + b < a.D) &&
                          take_mutant(w.w[b], j0 + b, jrand, crt);
          const float mv = mutant_coord(get(v1[p], b), get(v2[p], b),
                                        get(v3[p], b), Fr, a.lo, a.hi);
          const float u = tk ? mv : get(px[p], b);
          set(pu[p], b, u);
          set(y, b, (j0 + b < a.D) ? u - get(ov, b) : 0.f);
        }
        T* arow = At + (size_t)rl * stride;
        if (live && j0 < dpad) put_quad<P>(arow, j0, y);
      }
    }
  } else
  {
    // Chunk-major: for each 256-coordinate chunk, the wave's rows rl = wave
    // + kRotWaves * k go RB at a time: the target and donor chunks of the RB
    // rows are requested together, then drawn, mutated and stored.  Rows are
    // scalar and the chunk's groups q per lane, so the crossover draws share
    // their first rounds (XoverCol, XoverRow).  All workgroups
    // walk the chunks in the same order, so an XCD's donor reads of one
    // step stay within one chunk of its runs' rows (a working set its L2
    // holds).  Loads past the end of a row go to its last chunk and rows
    // past the wave's last go to its last row (values unused), so no load
    // sits behind a per-lane branch.
    const RotRows c{base, donors, ctl, planes, rng_run, row0, nvalid, stride,
                    tq};
    for (int t = 0; t < tq; ++t)
      build_chunk<P, sizeof(T) == 2 ? (BM / kRotWaves < kBf16Rows
                                           ? BM / kRotWaves
                                           : kBf16Rows)
                                    : (BM / kRotWaves < 8 ? BM / kRotWaves : 8),
                  kRotWaves, EVAL, JDE>(a, c, t, At);
  }
  __syncthreads();

  SelectRow sr{0, false, 0.f, false};
  if constexpr (!PAIR)
    sr = select_row<kRotWaves, EVAL>(a, run, row0, nvalid);

  // ---- phase 2: Z = Y R^T with the objective fused into the epilogue
  // Accumulators c{m}{n}: 32x32 block (row block m, column block nb0 + n),
  // named values rather than arrays so that every index is static.
  // Wave w of every workgroup streams the same R fragments at about the same
  // time, so concurrent requests from the CUs of an XCD share L2 lines.
  const int nblk = dpad / 32;
  // Row sums of the objective go to kRotSlots slots: slot s adds column
  // blocks s, s + 16, s + 32, ... in increasing order, so the result does
  // not depend on how blocks are dealt to waves (the number of threads).
  // A wave's blocks fall into SPW slots, its pass p into sacc[p % SPW].
  constexpr int SPW = kRotSlots / kRotWaves > 1 ? kRotSlots / kRotWaves : 1;
  static_assert(kRotSlots % kRotWaves == 0, "slots and waves");
  float sacc[SPW];
#pragma unroll
  for (int q = 0; q < SPW; ++q) sacc[q] = 0.f;
  int pass = 0;
  for (int nb0 = wave; nb0 < nblk; nb0 += kRotWaves, ++pass) {
    floatx16 c00 = {}, c01 = {}, c10 = {};
    if constexpr (P::kParts == 3) {
      floatx16 acc[1][1] = {{c00}};
      const int kbn = dpad / 16;
      x3_product<1, 1>(acc,
                       At + (size_t)(lane % 32) * stride + 24 * (lane / 32), 0,
                       reinterpret_cast<const float4*>(a.rop) +
                           (size_t)__builtin_amdgcn_readfirstlane(nb0) * kbn *
                               128,
                       0, (a.D + 15) / 16, lane, 1);
      c00 = acc[0][0];
    } else if constexpr (sizeof(T) == 2) {
      // R as [nblk][dpad/16][64 lanes][8]: one 16-byte load per lane per
      // block and K-step; dpad / 16 is a multiple of 8.
      // Software pipeline at K-step granularity: the A fragments of step
      // k + 1 are read from LDS while step k's MFMAs run (two slots), and
      // step k's registers of R fragments are loaded for step k + 8 once its
      // MFMAs are issued.  No load is behind a branch (the last group loads
      // itself again) and the first eight keep the loop's order (barriers):
      // otherwise the compiler cannot count the loads in flight and waits
      // for all of them at the loop's head, an L2 round trip per eight steps.
      const int kbn = dpad / 16;
      const bf16x8* rbu = reinterpret_cast<const bf16x8*>(a.rop) +
                          (size_t)__builtin_amdgcn_readfirstlane(nb0) * kbn * 64;
      const T* ar = At + (size_t)(lane % 32) * stride + 8 * (lane / 32);
      const T* ar1 = ar + (size_t)32 * stride;
      bf16x8 a0s[2], a1s[2], bf[8];
      a0s[0] = *reinterpret_cast<const bf16x8*>(ar);
      if constexpr (MB == 2) a1s[0] = *reinterpret_cast<const bf16x8*>(ar1);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        bf[u] = rbu[u * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
      }
      for (int kb = 0; kb < kbn; kb += 8) {
        const int kn = kb + 8 < kbn ? kb + 8 : kb;
        const bf16x8* rbn = rbu + (size_t)kn * 64;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int cur = u & 1, nxt = cur ^ 1;
          const int ka = u < 7 ? kb + u + 1 : kn;
          a0s[nxt] = *reinterpret_cast<const bf16x8*>(ar + ka * 16);
          if constexpr (MB == 2)
            a1s[nxt] = *reinterpret_cast<const bf16x8*>(ar1 + ka * 16);
          c00 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0s[cur], bf[u], c00,
                                                        0, 0, 0);
          if constexpr (MB == 2) {
            c10 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1s[cur], bf[u], c10,
                                                          0, 0, 0);
          }
          bf[u] = rbn[u * 64 + lane];
          interleave_step<MB>();
        }
      }
    } else {
      // R as [nblk][dpad/8][64 lanes][4]: one float4 = four K-steps; dpad / 8
      // is a multiple of 2.  Even and odd four-step groups accumulate apart
      // (two independent MFMA chains), then add.
      const float4* rop = reinterpret_cast<const float4*>(a.rop);
      const int k8n = dpad / 8;
      const float4* rb0 = rop + ((size_t)nb0 * k8n) * 64 + lane;
      const float* ar = reinterpret_cast<const float*>(At) +
                        (size_t)(lane % 32) * stride + 4 * (lane / 32);
      float4 p0 = rb0[0], p1 = rb0[64];
      for (int k8 = 0; k8 < k8n; k8 += 2) {
        const float4 q0 = p0, q1 = p1;
        if (k8 + 2 < k8n) {
          const size_t nx = (size_t)(k8 + 2) * 64;
          p0 = rb0[nx];
          p1 = rb0[nx + 64];
        }
        f32_step2(ar, k8, q0, q1, c00, c01);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) c00[r] += c01[r];
    }
    // The objective of each 32-column block, summed per row and written to
    // the block's LDS slot; rows then add the slots in block order, so the
    // result does not depend on how blocks are dealt to waves (the number
    // of threads).  32x32 accumulator layout: register r of lane l holds
    // row 8 (r / 4) + 4 (l / 32) + r % 4 and column l % 32 of the block.
    // Each lane has 16 values of one row block, or 32 of two; a
    // reduce-scatter butterfly over the 32 lanes of each half-wave leaves
    // lane l with the total of value l % 32 (31 exchanges instead of 5 per
    // value).
    constexpr bool kFastSin = sizeof(T) == 2 && P::kParts == 1;
    constexpr bool kHi = MB == 2;
    const floatx16& lo = c00;
    const floatx16& hi = MB == 2 ? c10 : c01;
    const float total = osc_rows<kFastSin, kHi>(lo, hi, lane);
#pragma unroll
    for (int q = 0; q < SPW; ++q)
      if (pass % SPW == q) sacc[q] += total;
  }
  // lane l holds value l % 32: row (l % 32 / 16) * 32 + rin of the wave's
  // blocks (one row block: the lanes with l % 32 < 16)
  {
    const int idx = lane % 32, hb = idx / 16, r = idx % 16;
    const int rin = 8 * (r / 4) + 4 * (lane / 32) + (r % 4);
#pragma unroll
    for (int q = 0; q < SPW; ++q) {
      const int b0 = wave + q * kRotWaves;  // first block of q
      if ((MB == 2 || hb == 0) && b0 < kRotSlots)
        fpart[(size_t)b0 * BM + hb * 32 + rin] = sacc[q];
    }
  }
  __syncthreads();

  // ---- phase 3: selection and the next generation
  if constexpr (PAIR) {
    // two rows per wave instruction as in the build, from the registers it
    // left; lanes 0 and 32 each write their row's value, flag and statistics
    const int nrow_w = wave < nvalid ? (nvalid - 1 - wave) / kRotWaves + 1 : 0;
    const int j0 = 4 * ql;
#pragma unroll
    for (int p = 0; p < RBP; ++p) {
      const int kk = 2 * p + hl;
      if (kk >= nrow_w) continue;
      const int rl = wave + kRotWaves * kk;
      float f = 0.f;
#pragma unroll
      for (int sl = 0; sl < kRotSlots; ++sl) f += fpart[sl * BM + rl];
      const int i = row0 + rl;
      const size_t g = (size_t)run * a.NP + i;
      const float fx = pf[p];
      const bool accept = f < fx;
      if ((accept || pchg[p]) && j0 < a.D) {
        float4 out;
#pragma unroll
        for (int b = 0; b < 4; ++b)
          set(out, b, accept ? get(pu[p], b) : get(px[p], b));
        st4(a.pop_next + g * a.ldx + j0, out);
      }
      if (ql == 0) {
        a.fit_next[g] = accept ? f : fx;
        a.changed[g] = accept ? 1 : 0;
        if constexpr (JDE) {
          // the trial's F', CR' survive only with the trial
          a.jp_next[g] = accept ? make_float2(ctl[rl].F, ctl[rl].CR)
                                : a.jp_cur[g];
        }
        if (accept) record_accept(a, run, i, f);
      }
    }
    return;
  }
  const RotRows c{base, donors, ctl, planes, rng_run, row0, nvalid, stride, tq};
  select_rows<BM, kRotWaves, EVAL, JDE>(a, c, run, fpart, sr);
}

// ---------------------------------------------------------------------------
// FP32 tile of three-part operands for rows of more than 128 coordinates, and
// for evaluations: 32 MB rows, NW waves.  The A tile holds kX3Part coordinates
// at a time (six bytes each: whole rows of 1000 would not fit); the next part
// is built when the product of the last is done, and every wave keeps z of its
// column blocks wave, wave + NW, ... (at most NB) over the parts.  Every form
// adds the same numbers in the same order, so a value does not depend on which
// one computed it.
constexpr int kX3Part = 256;

__host__ __device__ constexpr size_t x3_lds_bytes(int bm, int dpad, bool jde) {
  const int tq = (dpad / 4 + 63) / 64;
  return (size_t)bm * (3 * kX3Part + PrecX3::kPad) * sizeof(__bf16)  // A tile
         + (size_t)bm * tq * 4 * sizeof(unsigned long long)          // planes
         + (size_t)bm * 4 * sizeof(int)                              // donors
         + (size_t)kRotSlots * bm * sizeof(float)                    // slot sums
         + (jde ? (size_t)bm * sizeof(Control) : 0);                 // F', CR'
}

template <int MB, int NB, int NW, bool EVAL, bool JDE>
__device__ __forceinline__ void rot_tile_x3(const GenArgs& a, int run, int row0,
                                            int nvalid) {
  constexpr int BM = 32 * MB;
  static_assert(NW == 8 || NW == 16, "slots and waves");
  extern __shared__ __align__(16) char smem[];
  const int stride = 3 * kX3Part + PrecX3::kPad;
  const int tq = (a.dpad / 4 + 63) / 64;
  __bf16* At = reinterpret_cast<__bf16*>(smem);
  unsigned long long* planes =
      reinterpret_cast<unsigned long long*>(At + (size_t)BM * stride);
  int* donors = reinterpret_cast<int*>(planes + (size_t)BM * tq * 4);
  float* fpart = reinterpret_cast<float*>(donors + BM * 4);
  Control* ctl = reinterpret_cast<Control*>(fpart + kRotSlots * BM);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int lane = (int)threadIdx.x % 64;
  const uint32_t rng_run = a.run_base + (uint32_t)run;
  const RotRows c{a.pop_cur + (EVAL ? 0 : (size_t)run * a.NP * a.ldx),
                  donors, ctl, planes, rng_run, row0, nvalid, stride, tq};
  if (!EVAL) {
    if ((int)threadIdx.x < nvalid) {
      const int rl = (int)threadIdx.x;
      const Donors d = pick_donors(rng_run, a.gen, row0 + rl, a.NP, a.D,
                                   a.key_lo, a.key_hi);
      donors[rl * 4 + 0] = d.r1;
      donors[rl * 4 + 1] = d.r2;
      donors[rl * 4 + 2] = d.r3;
      donors[rl * 4 + 3] = d.jrand;
      if constexpr (JDE) {
        const float2 p = a.jp_cur[(size_t)run * a.NP + row0 + rl];
        ctl[rl] = jde_control(rng_run, a.gen, row0 + rl, a.key_lo, a.key_hi,
                              a.jF_lo, a.jF_span, a.jtau_F, a.jtau_CR,
                              Control{p.x, p.y});
      }
    }
    __syncthreads();
  }
  const SelectRow sr = select_row<NW, EVAL>(a, run, row0, nvalid);
  // column blocks past D hold zeros: left out, like the K-steps past D
  const int nblk = (a.D + 31) / 32, kbn = a.dpad / 16;
  const int mine = wave < nblk ? (nblk - 1 - wave) / NW + 1 : 0;
  floatx16 acc[NB][MB];
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[n][m] = floatx16{};
  const float4* rb = reinterpret_cast<const float4*>(a.rop) +
                     (size_t)(wave < nblk ? wave : 0) * kbn * 128;
  const size_t bstep = (size_t)NW * kbn * 128;
  const __bf16* ar = At + (size_t)(lane % 32) * stride + 24 * (lane / 32);
  for (int t = 0; t < tq; ++t) {
    if (t > 0) __syncthreads();  // the last part's products are done
    // rows past the tile's last keep what the LDS held: their sums are unused
    build_chunk<PrecX3, (MB == 2 ? 2 : BM / NW), NW, EVAL, JDE>(
        a, c, t, At - 3 * kX3Part * t);
    __syncthreads();
    const int steps = (min(kX3Part, a.D - kX3Part * t) + 15) / 16;
    const float4* rt = rb + (size_t)t * (kX3Part / 16) * 128;
    if (mine > 0)
      x3_product<MB, NB>(acc, ar, 32 * stride, rt, bstep, steps, lane, mine);
  }
  // row sums of the objective: block b goes to slot b mod 16, a slot's blocks
  // in order
  float sacc[2] = {0.f, 0.f};
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const float total = osc_rows<false, MB == 2>(acc[n][0], acc[n][MB - 1], lane);
    if (n < mine) sacc[NW == 8 ? n & 1 : 0] += total;
  }
  {
    const int idx = lane % 32, hb = idx / 16, r = idx % 16;
    const int rin = 8 * (r / 4) + 4 * (lane / 32) + (r % 4);
    if (MB == 2 || hb == 0) {
      fpart[(size_t)wave * BM + hb * 32 + rin] = sacc[0];
      if (NW == 8) fpart[(size_t)(wave + 8) * BM + hb * 32 + rin] = sacc[1];
    }
  }
  __syncthreads();
  select_rows<BM, NW, EVAL, JDE>(a, c, run, fpart, sr);
}

}  // namespace de

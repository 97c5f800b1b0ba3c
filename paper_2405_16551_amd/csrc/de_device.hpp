// de_device.hpp -- device-side building blocks of the gfx950 DE/rand/1/bin
// kernels: counter-based random draws, the donor sampler of eq. 2, the
// crossover test of eq. 3, bound repair, ordered (f, index) keys and
// wave64 reductions.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11).  The
// 128-bit counter is (q, i, gen, tag << 24 | run) and the key is the 64-bit
// seed, so every draw is a pure function of its coordinates and no
// generator state lives in memory.  Integer-only conversions keep every
// index and every crossover decision independent of floating point.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace de {

enum : uint32_t {
  kTagInit = 1u,
  kTagIdx = 2u,
  kTagXover = 3u,
  kTagJde = 4u,
  kTagTrain = 5u,   // surrogate: minibatch rows
  kTagModel = 6u    // surrogate: initial weights
};

// Philox4x32-10 multipliers and Weyl key increments (Salmon et al., Sec. 4).
constexpr uint32_t kPhiloxMulA = 0xD2511F53u;
constexpr uint32_t kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kPhiloxWeylA = 0x9E3779B9u;
constexpr uint32_t kPhiloxWeylB = 0xBB67AE85u;

struct Words4 {
  uint32_t w[4];
};

// Three-way XOR; on gfx950 one v_bitop3_b32 (truth table 0x96) instead of
// two v_xor_b32.
__host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b,
                                                  uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}

// One S-box round: two 32x32->64 products (v_mad_u64_u32 on CDNA), the
// high halves mixed with the other two counter words and the round key.
__host__ __device__ __forceinline__ void philox_round(uint32_t& c0, uint32_t& c1,
                                             uint32_t& c2, uint32_t& c3,
                                             uint32_t k0, uint32_t k1) {
  const uint64_t pa = (uint64_t)kPhiloxMulA * c0;
  const uint64_t pb = (uint64_t)kPhiloxMulB * c2;
  const uint32_t n0 = xor3((uint32_t)(pb >> 32), c1, k0);
  const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
  c1 = (uint32_t)pb;
  c3 = (uint32_t)pa;
  c0 = n0;
  c2 = n2;
}

__host__ __device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1,
                                                uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    philox_round(c0, c1, c2, c3, k0 + (uint32_t)r * kPhiloxWeylA,
                 k1 + (uint32_t)r * kPhiloxWeylB);
  }
  Words4 out;
  out.w[0] = c0;
  out.w[1] = c1;
  out.w[2] = c2;
  out.w[3] = c3;
  return out;
}

// Draw block for (tag, run, gen, individual, group q).
__host__ __device__ __forceinline__ Words4 draw_block(uint32_t tag, uint32_t run,
                                             uint32_t gen, uint32_t indiv,
                                             uint32_t q, uint32_t key_lo,
                                             uint32_t key_hi) {
  return philox4x32_10(q, indiv, gen, (tag << 24) | run, key_lo, key_hi);
}

// Crossover blocks draw_block(kTagXover, run, gen, i, q) of many rows i and
// groups q, with what rounds 1 to 3 owe to q alone (XoverCol) and to i alone
// (XoverRow) computed once: of the 20 products of a block 15 are left where
// a wave walks rows i (scalar) at fixed q (per lane), and the trial build
// spends a third of its vector instructions on them.
struct XoverCol {
  uint32_t n3, m1, h2, l2;
};
struct XoverRow {
  uint32_t h1, l1;
};

__host__ __device__ __forceinline__ XoverCol xover_col(uint32_t run,
                                                       uint32_t gen, uint32_t q,
                                                       uint32_t k0,
                                                       uint32_t k1) {
  const uint32_t n1 = kPhiloxMulB * gen;
  const uint64_t pa0 = (uint64_t)kPhiloxMulA * q;
  const uint32_t n2 = xor3((uint32_t)(pa0 >> 32), (kTagXover << 24) | run, k1);
  const uint64_t pb1 = (uint64_t)kPhiloxMulB * n2;
  const uint32_t m0 = xor3((uint32_t)(pb1 >> 32), n1, k0 + kPhiloxWeylA);
  const uint64_t pa2 = (uint64_t)kPhiloxMulA * m0;
  XoverCol c;
  c.n3 = (uint32_t)pa0;
  c.m1 = (uint32_t)pb1 ^ (k0 + 2u * kPhiloxWeylA);
  c.h2 = (uint32_t)(pa2 >> 32) ^ (k1 + 2u * kPhiloxWeylB);
  c.l2 = (uint32_t)pa2;
  return c;
}

__host__ __device__ __forceinline__ XoverRow xover_row(uint32_t gen,
                                                       uint32_t indiv,
                                                       uint32_t k0,
                                                       uint32_t k1) {
  const uint64_t pb0 = (uint64_t)kPhiloxMulB * gen;
  const uint64_t pa1 =
      (uint64_t)kPhiloxMulA * xor3((uint32_t)(pb0 >> 32), indiv, k0);
  return {(uint32_t)(pa1 >> 32) ^ (k1 + kPhiloxWeylB), (uint32_t)pa1};
}

__host__ __device__ __forceinline__ Words4 xover_words(XoverCol c, XoverRow r,
                                                       uint32_t k0,
                                                       uint32_t k1) {
  const uint64_t pb2 = (uint64_t)kPhiloxMulB * (r.h1 ^ c.n3);
  uint32_t c0 = (uint32_t)(pb2 >> 32) ^ c.m1, c1 = (uint32_t)pb2;
  uint32_t c2 = c.h2 ^ r.l1, c3 = c.l2;
#pragma unroll
  for (int n = 3; n < 10; ++n)
    philox_round(c0, c1, c2, c3, k0 + (uint32_t)n * kPhiloxWeylA,
                 k1 + (uint32_t)n * kPhiloxWeylB);
  return {{c0, c1, c2, c3}};
}

// Uniform integer in [0, n) from one 32-bit word: floor(w * n / 2^32).
__host__ __device__ __forceinline__ int uniform_below(uint32_t w, uint32_t n) {
  return (int)(((uint64_t)w * n) >> 32);
}

// Donor triple and j_rand of eq. 2 / eq. 3 for target i.  a, b, c are
// uniform over NP-1, NP-2, NP-3 values; each is lifted over the indices
// already taken (target first, then earlier donors), in ascending order, so
// (a, b, c) maps one-to-one onto ordered triples of distinct indices != i.
struct Donors {
  int r1, r2, r3, jrand;
};

// From the words of the individual's IDX block; i is the target to avoid.
__host__ __device__ __forceinline__ Donors donors_of(const Words4& w, int i,
                                                     int NP, int D) {
  Donors d;
  const int a = uniform_below(w.w[0], (uint32_t)(NP - 1));
  d.r1 = a + (a >= i ? 1 : 0);
  const int lo2 = min(i, d.r1), hi2 = max(i, d.r1);
  int b = uniform_below(w.w[1], (uint32_t)(NP - 2));
  b += (b >= lo2 ? 1 : 0);
  b += (b >= hi2 ? 1 : 0);
  d.r2 = b;
  // ascending order of {i, r1, r2}
  int s0 = lo2, s1 = hi2, s2 = b;
  if (s2 < s1) { const int t = s1; s1 = s2; s2 = t; }
  if (s1 < s0) { const int t = s0; s0 = s1; s1 = t; }
  int c = uniform_below(w.w[2], (uint32_t)(NP - 3));
  c += (c >= s0 ? 1 : 0);
  c += (c >= s1 ? 1 : 0);
  c += (c >= s2 ? 1 : 0);
  d.r3 = c;
  d.jrand = uniform_below(w.w[3], (uint32_t)D);
  return d;
}

// ctr_i is the counter's individual field (i itself, or i | c << 24 for
// candidate c of the surrogate-assisted step).
__host__ __device__ __forceinline__ Donors pick_donors_ctr(
    uint32_t run, uint32_t gen, uint32_t ctr_i, int i, int NP, int D,
    uint32_t key_lo, uint32_t key_hi) {
  return donors_of(draw_block(kTagIdx, run, gen, ctr_i, 0u, key_lo, key_hi), i,
                   NP, D);
}

__host__ __device__ __forceinline__ Donors pick_donors(uint32_t run, uint32_t gen,
                                              int i, int NP, int D,
                                              uint32_t key_lo,
                                              uint32_t key_hi) {
  return pick_donors_ctr(run, gen, (uint32_t)i, i, NP, D, key_lo, key_hi);
}

// Crossover test of eq. 3 for coordinate j = 4q + b: rand_j = (w >> 8) 2^-24
// and rand_j <= CR  <=>  (w >> 8) <= floor(CR 2^24) = cr_threshold
// <=>  w <= 256 cr_threshold + 255 (all words when cr_threshold >= 2^24 - 1),
// one comparison of the whole word.  The limit depends on the threshold
// only, so loops compute it once.
__host__ __device__ __forceinline__ uint32_t xover_word_limit(
    uint32_t cr_threshold) {
  return cr_threshold >= 0xFFFFFFu ? 0xFFFFFFFFu
                                   : (cr_threshold << 8) | 0xFFu;
}

__host__ __device__ __forceinline__ bool take_mutant(uint32_t word, int j, int jrand,
                                            uint32_t cr_threshold) {
  return (j == jrand) | (word <= xover_word_limit(cr_threshold));
}

// Mutant coordinate of eq. 2 with clamping to the box; NaN passes through
// (on gfx950 as v_maximum3 / v_minimum3, which hand a NaN on, instead of two
// compares and two selects with their wait states: 16 x 1024 x 1000 sphere 386
// us per 20 generations against 401, BF16 1143 / 1168).  Of a zero and a bound
// of zero with unlike signs maximum takes +0 and minimum -0 where the selects
// keep the coordinate: -0, which only a loaded row can hold, becomes +0 at lo =
// +0.  The two compare equal and give the same f.
__host__ __device__ __forceinline__ float mutant_coord(float x1, float x2, float x3,
                                              float F, float lo, float hi) {
  float v = fmaf(F, x2 - x3, x1);
#if defined(__HIP_DEVICE_COMPILE__)
  v = __builtin_elementwise_minimum(__builtin_elementwise_maximum(v, lo), hi);
#else
  v = v < lo ? lo : v;
  v = v > hi ? hi : v;
#endif
  return v;
}

// jDE control values of individual i for this generation (self-adaptation
// of Brest et al., 2006): one Philox block (tag 4, group 0) gives u1..u4 on
// the 2^-24 lattice; F' = F_lo + u1 F_span (one fused rounding) if
// u2 < tau_F, else the stored F; CR' = u3 if u4 < tau_CR, else the stored
// CR.  tau thresholds are floor(tau 2^24), compared in integers.
struct Control {
  float F, CR;
};

__host__ __device__ __forceinline__ Control jde_control(
    uint32_t run, uint32_t gen, int i, uint32_t key_lo, uint32_t key_hi,
    float F_lo, float F_span, uint32_t tau_F, uint32_t tau_CR, Control cur) {
  const Words4 w = draw_block(kTagJde, run, gen, (uint32_t)i, 0u, key_lo,
                              key_hi);
  Control c = cur;
  if ((w.w[1] >> 8) < tau_F)
    c.F = fmaf((float)(w.w[0] >> 8) * 0x1.0p-24f, F_span, F_lo);
  if ((w.w[3] >> 8) < tau_CR) c.CR = (float)(w.w[2] >> 8) * 0x1.0p-24f;
  return c;
}

// floor(CR 2^24) for a float CR in [0, 1] (the scaling is exact).
__host__ __device__ __forceinline__ uint32_t cr_threshold_of(float CR) {
  return (uint32_t)(CR * 16777216.0f);
}

// Totally ordered 64-bit key: order-preserving image of the float in the high
// half (NaN sorts above +inf), individual index in the low half, so
// atomicMin yields the lowest value with ties to the lowest index.
__host__ __device__ __forceinline__ unsigned long long fit_key(float f, int idx) {
  const uint32_t b = __builtin_bit_cast(uint32_t, f);
  const uint32_t ord = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((unsigned long long)ord << 32) | (uint32_t)idx;
}

// sin^2(t), t in FP32.  t = k (pi/2) + r with |r| <= pi/4: k = rint(t 2/pi),
// r by Cody-Waite reduction with pi/2 split into three FP32 parts (each
// product k * part folded in with one FMA).  sin^2(t) = sin^2(r) for even k
// and 1 - sin^2(r) for odd k.  sin^2(r) from its Taylor series
// sum_{n>=1} (-1)^(n+1) 2^(2n-1) r^(2n) / (2n)!, six terms: the first
// omitted term is below 4e-9 on |r| <= pi/4, under half an FP32 ulp of 0.5.
__host__ __device__ __forceinline__ float sin_squared(float t) {
  constexpr float kTwoOverPi = 0x1.45f306p-1f;
  constexpr float kHalfPiA = 0x1.921fb6p+0f;
  constexpr float kHalfPiB = -0x1.777a5cp-25f;
  constexpr float kHalfPiC = -0x1.ee59dap-50f;
  const float k = rintf(t * kTwoOverPi);
  float r = fmaf(-k, kHalfPiA, t);
  r = fmaf(-k, kHalfPiB, r);
  r = fmaf(-k, kHalfPiC, r);
  const float s = r * r;
  float p = -2.0f / 467775.0f;
  p = fmaf(p, s, 2.0f / 14175.0f);
  p = fmaf(p, s, -1.0f / 315.0f);
  p = fmaf(p, s, 2.0f / 45.0f);
  p = fmaf(p, s, -1.0f / 3.0f);
  p = fmaf(p, s, 1.0f);
  p *= s;
  return ((int)k & 1) ? 1.0f - p : p;
}

#if defined(__HIPCC__)
// v of lane l ^ m, for m = 1, 2, 4, 8 within a row of 16 lanes by data-parallel
// moves (a few clocks instead of an LDS round trip), 16 and 32 through the
// LDS crossbar.
template <int ctrl>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl,
                                         0xF, 0xF, true));
}

template <int m>
__device__ __forceinline__ float lane_xor(float v) {
  if constexpr (m == 1) return dpp_move<0xB1>(v);   // quad 1 0 3 2
  if constexpr (m == 2) return dpp_move<0x4E>(v);   // quad 2 3 0 1
  if constexpr (m == 4) return dpp_move<0x1B>(dpp_move<0x141>(v));  // 7-l, 3-l
  if constexpr (m == 8) return dpp_move<0x128>(v);  // row rotated by 8
  if constexpr (m == 16)
    return __builtin_bit_cast(
        float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
  return __shfl_xor(v, m, 64);
}

// Sum over aligned groups of `width` lanes (power of two <= 64) by
// butterfly exchange; every lane of the group ends with the same total, and
// the order of additions is fixed.
template <int width>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (width >= 64) v += lane_xor<32>(v);
  if constexpr (width >= 32) v += lane_xor<16>(v);
  if constexpr (width >= 16) v += lane_xor<8>(v);
  if constexpr (width >= 8) v += lane_xor<4>(v);
  if constexpr (width >= 4) v += lane_xor<2>(v);
  if constexpr (width >= 2) v += lane_xor<1>(v);
  return v;
}
#endif

// Block index remapping so that consecutive logical blocks land on the same
// XCD (gfx950 dispatches block b to XCD b mod 8): logical block ranges, and
// the donor rows they share, then stay in one XCD's L2.  Bijective for any n.
__host__ __device__ __forceinline__ int xcd_logical_block(int b, int n) {
  constexpr int kXcd = 8;
  const int q = n / kXcd, r = n % kXcd;
  const int xcd = b % kXcd, k = b / kXcd;
  return xcd * q + min(xcd, r) + k;
}

}  // namespace de

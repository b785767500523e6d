// device_math.h -- device-side primitives of the decoder: the counter-based
// generator behind every random draw, and the FP32 arithmetic of the BP
// check rule (BP-LLR2). Compiled with -ffp-contract=off: every expression
// below is one IEEE operation per arithmetic operator (fmaf one fused
// operation), evaluated in the order written, so results are reproducible
// bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace laim {

// Work-item and work-group indices, the work-group size, and the high half
// of a 32-bit product, from the compiler's builtins. The kernels are built
// with IEEE mode off (-mno-amdgpu-ieee); the device library behind
// threadIdx, blockIdx, blockDim and __umulhi is not, so its accessors would
// not be inlined (their floating-point modes differ) and every use would be
// a function call.
__device__ __forceinline__ uint32_t tid_x() { return __builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ uint32_t bid_x() { return __builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ uint32_t bid_y() { return __builtin_amdgcn_workgroup_id_y(); }
__device__ __forceinline__ uint32_t bdim_x() { return __builtin_amdgcn_workgroup_size_x(); }
__device__ __forceinline__ uint32_t mulhi_u32(uint32_t a, uint32_t b) {
  return (uint32_t)(((uint64_t)a * (uint64_t)b) >> 32);
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw: "Parallel random numbers: as
// easy as 1, 2, 3", SC'11). Ten rounds of the 4x32 S-box: the products of
// words 0 and 2 with the two round multipliers are split into halves; the
// high halves are mixed into words 1 and 3 together with the round key;
// the round key advances by the two Weyl constants after each round.
struct Philox4 {
  uint32_t w0, w1, w2, w3;
};

__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const uint32_t a = 0xD2511F53u * c0;                  // low half of M0 * c0
    const uint32_t ah = mulhi_u32(0xD2511F53u, c0);        // high half
    const uint32_t b = 0xCD9E8D57u * c2;
    const uint32_t bh = mulhi_u32(0xCD9E8D57u, c2);
    const uint32_t n0 = bh ^ c1 ^ k0;
    const uint32_t n2 = ah ^ c3 ^ k1;
    c0 = n0;
    c1 = b;
    c2 = n2;
    c3 = a;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Philox4{c0, c1, c2, c3};
}

// Bernoulli event "w < bound" with a 64-bit bound (bound = 2^32 means always).
__device__ __forceinline__ bool below(uint32_t w, uint64_t bound) { return (uint64_t)w < bound; }

__device__ __forceinline__ float clampf(float x, float c) { return fminf(fmaxf(x, -c), c); }

// Smallest of three (exact; the compiler forms one v_min3_f32).
__device__ __forceinline__ float min3f(float a, float b, float c) { return fminf(fminf(a, b), c); }

// min(|a|, |b|, |c|) as a single v_min3_f32. Written as an asm statement so
// that the compiler cannot split several of them into two-input minima
// shared between results, which costs one more instruction per four.
// Exact, and equal to min3f(fabsf(a), fabsf(b), fabsf(c)) for non-NaN input.
__device__ __forceinline__ float min3_abs(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// ex[j] = the smallest |x[i]| over i != j, exactly (a minimum rounds nothing, so
// any grouping gives the same value). Checks of degree 6 and 8 take the minima
// of pairs, and of pairs of pairs, and one three-input minimum per output: 9
// and 14 instructions against 12 and 18 for prefix and suffix minima.
template <int DC>
__device__ __forceinline__ void min_others(const float* x, float* ex) {
  if constexpr (DC == 2) {
    ex[0] = fabsf(x[1]);
    ex[1] = fabsf(x[0]);
  } else if constexpr (DC == 4) {
    ex[0] = min3_abs(x[1], x[2], x[3]);
    ex[1] = min3_abs(x[0], x[2], x[3]);
    ex[2] = min3_abs(x[0], x[1], x[3]);
    ex[3] = min3_abs(x[0], x[1], x[2]);
  } else {
    static_assert(DC == 6 || DC == 8, "compiled check degrees");
    float p[DC / 2];
#pragma unroll
    for (int i = 0; i < DC / 2; ++i) p[i] = fminf(fabsf(x[2 * i]), fabsf(x[2 * i + 1]));
#pragma unroll
    for (int i = 0; i < DC / 2; ++i) {
      // the other pairs' minimum: two pairs as they are (degree 6), or the
      // pair beside this one and the two of the other half (degree 8)
      const float a = DC == 6 ? p[(i + 1) % 3] : p[i ^ 1];
      const float b = DC == 6 ? p[(i + 2) % 3] : fminf(p[(i & 2) ^ 2], p[((i & 2) ^ 2) + 1]);
      ex[2 * i] = min3_abs(x[2 * i + 1], a, b);
      ex[2 * i + 1] = min3_abs(x[2 * i], a, b);
    }
  }
}

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// e^x for x <= 0, by Cody-Waite reduction x = k ln2 + r (ln2 split into a
// head with 16 significant bits, so k*head is exact, and a tail), the
// degree-7 Taylor polynomial of e^r in Horner form with one fused
// multiply-add (a single rounding) per step, and a scale by 2^k: k, read off
// the low bits of k + 1.5 2^23, is added to the exponent field (exact: for
// x >= -80 the result is a normal number). Arguments below -80 (and -inf)
// give 0: what the sequence makes of them is not used, so no lane diverges.
//
// log(1 + u) for u in [0, 1] as u Q(u), Q the degree-9 polynomial that
// interpolates log(1 + u)/u at the 10 Chebyshev nodes of [0, 1] (computed in
// high precision, coefficients rounded to FP32), in Horner form with one
// fused multiply-add per step: no division, under 3 ulp of relative error.
//
// Both are chains of dependent multiply-adds: a wavefront alone issues such a
// chain at one instruction in 10.7 clocks, two interleaved chains at one in
// 7.3 and four at one in 5.8, and four wavefronts per SIMD issue 7% more with
// four chains. The compiler schedules the chains one after another (it
// minimises registers), so N chains are interleaved here in asm statements,
// one instruction of each in turn. They read and write vector registers
// only, and read one scalar constant.
#define LAIM_X1(I) I(0)
#define LAIM_X2(I) I(0) I(1)
#define LAIM_X3(I) I(0) I(1) I(2)
#define LAIM_X4(I) I(0) I(1) I(2) I(3)

// Stage 1: t = floor(x log2e + 1/2), kb = t + 1.5 2^23, p = e^r's polynomial.
#define LAIM_E0(i) "v_fma_f32 %[t" #i "], %[x" #i "], %[l], 0.5\n\t"
#define LAIM_E1(i) "v_floor_f32 %[t" #i "], %[t" #i "]\n\t"
#define LAIM_E2(i) "v_fmamk_f32 %[r" #i "], %[t" #i "], 0xbf317200, %[x" #i "]\n\t"  /* -ln2 head */
#define LAIM_E3(i) "v_add_f32 %[k" #i "], 0x4b400000, %[t" #i "]\n\t"               /* + 1.5 2^23 */
#define LAIM_E4(i) "v_fmamk_f32 %[r" #i "], %[t" #i "], 0xb5bfbe8e, %[r" #i "]\n\t"  /* -ln2 tail */
#define LAIM_E5(i) "v_fmamk_f32 %[t" #i "], %[r" #i "], 0x39500d01, %[c]\n\t"        /* 1/5040, 1/720 */
#define LAIM_E6(i) "v_fmaak_f32 %[t" #i "], %[t" #i "], %[r" #i "], 0x3c088889\n\t"  /* 1/120 */
#define LAIM_E7(i) "v_fmaak_f32 %[t" #i "], %[t" #i "], %[r" #i "], 0x3d2aaaab\n\t"  /* 1/24 */
#define LAIM_E8(i) "v_fmaak_f32 %[t" #i "], %[t" #i "], %[r" #i "], 0x3e2aaaab\n\t"  /* 1/6 */
#define LAIM_E9(i) "v_fma_f32 %[t" #i "], %[t" #i "], %[r" #i "], 0.5\n\t"
#define LAIM_EA(i) "v_fma_f32 %[t" #i "], %[t" #i "], %[r" #i "], 1.0\n\t"
#define LAIM_EXP(X)                                                                             \
  X(LAIM_E0) X(LAIM_E1) X(LAIM_E2) X(LAIM_E3) X(LAIM_E4) X(LAIM_E5) X(LAIM_E6) X(LAIM_E7)       \
  X(LAIM_E8) X(LAIM_E9) X(LAIM_EA) X(LAIM_EA)
// Stage 2: q = u Q(u).
#define LAIM_L0(i) "v_fmamk_f32 %[q" #i "], %[u" #i "], 0xbb502565, %[c]\n\t"        /* -0x1.a04acap-9 */
#define LAIM_L1(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0xbd66e804\n\t"  /* -0x1.cdd008p-5 */
#define LAIM_L2(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0x3dd7eef4\n\t"  /* 0x1.afdde8p-4 */
#define LAIM_L3(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0xbe1c5c84\n\t"  /* -0x1.38b908p-3 */
#define LAIM_L4(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0x3e495a18\n\t"  /* 0x1.92b430p-3 */
#define LAIM_L5(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0xbe7f812a\n\t"  /* -0x1.ff0254p-3 */
#define LAIM_L6(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0x3eaaa5eb\n\t"  /* 0x1.554bd6p-2 */
#define LAIM_L7(i) "v_fmaak_f32 %[q" #i "], %[q" #i "], %[u" #i "], 0xbeffffdc\n\t"  /* -0x1.ffffb8p-2 */
#define LAIM_L8(i) "v_fma_f32 %[q" #i "], %[q" #i "], %[u" #i "], 1.0\n\t"
#define LAIM_L9(i) "v_mul_f32 %[q" #i "], %[u" #i "], %[q" #i "]\n\t"
#define LAIM_LOG(X)                                                                             \
  X(LAIM_L0) X(LAIM_L1) X(LAIM_L2) X(LAIM_L3) X(LAIM_L4) X(LAIM_L5) X(LAIM_L6) X(LAIM_L7)       \
  X(LAIM_L8) X(LAIM_L9)
#define LAIM_EOUT(i) [t##i] "=&v"(t[i]), [r##i] "=&v"(r[i]), [k##i] "=&v"(kb[i])
#define LAIM_EIN(i) [x##i] "v"(x[i])
#define LAIM_LOUT(i) [q##i] "=&v"(o[i])
#define LAIM_LIN(i) [u##i] "v"(u[i])

// o[i] = log(1 + e^{x[i]}), x[i] <= 0, i < N <= 4.
template <int N>
__device__ __forceinline__ void softplus_nonpos(const float* x, float* o) {
  static_assert(N >= 1 && N <= 4, "one to four chains");
  const float log2e = (float)1.44269504088896340736;
  const float c6 = 1.0f / 720.0f, q8 = 0x1.402f4cp-6f;
  float t[N], r[N], kb[N], u[N];
  if constexpr (N == 1)
    asm(LAIM_EXP(LAIM_X1) : LAIM_EOUT(0) : LAIM_EIN(0), [l] "s"(log2e), [c] "v"(c6));
  else if constexpr (N == 2)
    asm(LAIM_EXP(LAIM_X2) : LAIM_EOUT(0), LAIM_EOUT(1) : LAIM_EIN(0), LAIM_EIN(1), [l] "s"(log2e), [c] "v"(c6));
  else if constexpr (N == 3)
    asm(LAIM_EXP(LAIM_X3)
        : LAIM_EOUT(0), LAIM_EOUT(1), LAIM_EOUT(2)
        : LAIM_EIN(0), LAIM_EIN(1), LAIM_EIN(2), [l] "s"(log2e), [c] "v"(c6));
  else
    asm(LAIM_EXP(LAIM_X4)
        : LAIM_EOUT(0), LAIM_EOUT(1), LAIM_EOUT(2), LAIM_EOUT(3)
        : LAIM_EIN(0), LAIM_EIN(1), LAIM_EIN(2), LAIM_EIN(3), [l] "s"(log2e), [c] "v"(c6));
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float v = __uint_as_float(__float_as_uint(t[i]) + (__float_as_uint(kb[i]) << 23));
    u[i] = (x[i] < -80.0f) ? 0.0f : v;
  }
  if constexpr (N == 1)
    asm(LAIM_LOG(LAIM_X1) : LAIM_LOUT(0) : LAIM_LIN(0), [c] "v"(q8));
  else if constexpr (N == 2)
    asm(LAIM_LOG(LAIM_X2) : LAIM_LOUT(0), LAIM_LOUT(1) : LAIM_LIN(0), LAIM_LIN(1), [c] "v"(q8));
  else if constexpr (N == 3)
    asm(LAIM_LOG(LAIM_X3)
        : LAIM_LOUT(0), LAIM_LOUT(1), LAIM_LOUT(2)
        : LAIM_LIN(0), LAIM_LIN(1), LAIM_LIN(2), [c] "v"(q8));
  else
    asm(LAIM_LOG(LAIM_X4)
        : LAIM_LOUT(0), LAIM_LOUT(1), LAIM_LOUT(2), LAIM_LOUT(3)
        : LAIM_LIN(0), LAIM_LIN(1), LAIM_LIN(2), LAIM_LIN(3), [c] "v"(q8));
}

// a [+] b = 2 atanh(tanh(a/2) tanh(b/2)) (the two-input sum-product check
// rule; Hagenauer, Offer, Papke 1996), through its exact rewriting on the
// magnitudes |a| [+] |b| = min + log(1 + e^{-(|a|+|b|)}) - log(1 + e^{-||a|-|b||}),
// a negative rounding set to +0, and the sign sg(a) sg(b) with sg(x) = -1
// iff x < 0 for a nonzero result (a zero result is +0). No input is -0 (sums
// that start at +0 or a nonzero prior, and results of this function), so
// sg() is the sign bit; adding +0 makes a zero result +0.
// FAR: min(|a|, |b|) >= kBoxFar, where the first logarithm, at most 2.06e-7
// (|a| + |b| >= 15.4), is under half an ulp of the minimum (2^-22 = 2.38e-7 in
// [4, 8), more above): the sum rounds to the minimum and is not formed.
// N pairs at once (N <= 4): o[i] = a[i] [+] b[i].
constexpr float kBoxFar = 7.7f;
template <bool FAR, int N>
__device__ __forceinline__ void boxplus(const float* a, const float* b, float* o) {
  float nd[N], ny[N], sd[N], sy[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    nd[i] = __uint_as_float(__float_as_uint(fabsf(a[i]) - fabsf(b[i])) | 0x80000000u);
    ny[i] = -fabsf(a[i]) - fabsf(b[i]);
  }
  if constexpr (FAR) {
    softplus_nonpos<N>(nd, sd);
  } else {
#pragma unroll
    for (int i = 0; i + 1 < N; i += 2) {
      const float x4[4] = {nd[i], ny[i], nd[i + 1], ny[i + 1]};
      float o4[4];
      softplus_nonpos<4>(x4, o4);
      sd[i] = o4[0];
      sy[i] = o4[1];
      sd[i + 1] = o4[2];
      sy[i + 1] = o4[3];
    }
    if constexpr (N & 1) {
      const float x2[2] = {nd[N - 1], ny[N - 1]};
      float o2[2];
      softplus_nonpos<2>(x2, o2);
      sd[N - 1] = o2[0];
      sy[N - 1] = o2[1];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float mn = fminf(fabsf(a[i]), fabsf(b[i]));
    const float mag = fmaxf((FAR ? mn : mn + sy[i]) - sd[i], 0.0f);
    const uint32_t sg = __float_as_uint(a[i]) ^ __float_as_uint(b[i]);
    o[i] = __uint_as_float((__float_as_uint(mag) & 0x7FFFFFFFu) | (sg & 0x80000000u)) + 0.0f;
  }
}
__device__ __forceinline__ float boxplus1(float a, float b) {
  float o;
  boxplus<false, 1>(&a, &b, &o);
  return o;
}

// The sum-product check rule's box-plus of all inputs but one, for every
// output: acc[j] = F_{j-1} [+] B_{j+1} with the ascending prefix folds
// F_k = F_{k-1} [+] x_k and the suffix folds B_k = x_k [+] B_{k+1}; an
// empty side is dropped ((+inf) [+] y is y with -0 made +0, i.e. y + 0).
// 3 (D - 2) box-plus steps in D - 2 stages of independent ones: stage S forms
// F_S, B_{D-1-S} and the outputs whose two folds the stages before it made
// (output j in stage max(j - 1, D - 2 - j) + 1: none, one or two a stage).
// LEAN: one step at a time, for kernels short of registers.
template <int D, bool FAR, int S, bool LEAN>
__device__ __forceinline__ void boxplus_stage(const float* x, float* F, float* B, float* acc) {
  if constexpr (S <= D - 2) {
    constexpr int hi = S, lo = D - 1 - S;  // this stage's outputs, from the middle stage on
    constexpr bool any = hi >= lo, both = hi > lo;
    constexpr int N = both ? 4 : any ? 3 : 2;
    float a[N], b[N], o[N];
    a[0] = F[S - 1];
    b[0] = x[S];
    a[1] = x[D - 1 - S];
    b[1] = B[D - S];
    if constexpr (any) {
      a[2] = F[hi - 1];
      b[2] = B[hi + 1];
    }
    if constexpr (both) {
      a[3] = F[lo - 1];
      b[3] = B[lo + 1];
    }
    if constexpr (LEAN) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        boxplus<FAR, 1>(a + i, b + i, o + i);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      boxplus<FAR, N>(a, b, o);
    }
    F[S] = o[0];
    B[D - 1 - S] = o[1];
    if constexpr (any) acc[hi] = o[2];
    if constexpr (both) acc[lo] = o[3];
    boxplus_stage<D, FAR, S + 1, LEAN>(x, F, B, acc);
  }
}
template <int D, bool FAR, bool LEAN>
__device__ __forceinline__ void boxplus_folds(const float* x, float* acc) {
  float F[D], B[D];
  F[0] = x[0] + 0.0f;
  B[D - 1] = x[D - 1] + 0.0f;
  boxplus_stage<D, FAR, 1, LEAN>(x, F, B, acc);
  acc[0] = B[1];
  acc[D - 1] = F[D - 2];
}

// The same, with FAR steps where they serve for every check that the
// wavefront evaluates. A fold of i inputs is at least min - ln(i) (each step
// takes off log(1 + e^{-d}) at most, ln 2 for two equal inputs), so inputs of
// at least kBoxFar + ln(D - 1) + 0.01 make every step FAR (a step's roundings
// are relative to its minimum, far below the 0.01). One compare and one
// branch per check; half of the exponentials go in 38% of the
// wavefront-checks of the 2D toric code L = 32 at p = 0.05, and in 71% of
// those of the [[144,12,12]] code at p = 0.03.
template <int D>
__device__ constexpr float box_far_bound() {
  constexpr float kLn[] = {0.0f, 0.0f, 0.0f, 0.694f, 1.099f, 1.387f, 1.610f, 1.792f, 1.946f};
  return kBoxFar + kLn[D] + 0.01f;
}
template <int D, bool LEAN = false>
__device__ __forceinline__ void boxplus_all(const float* x, float* acc) {
  float mn = fabsf(x[0]);
#pragma unroll
  for (int k = 1; k < D; ++k) mn = fminf(mn, fabsf(x[k]));
  if (D > 2 && __builtin_amdgcn_ballot_w64(mn < box_far_bound<D>()) == 0ull)
    boxplus_folds<D, true, LEAN>(x, acc);
  else
    boxplus_folds<D, false, LEAN>(x, acc);
}

// The check rule with a check on two neighbouring lanes (an even and an odd
// one), for launches that leave most of the device idle: each lane forms half of
// the D outputs and the folds that they need. The even lane works on
// y_j = x_j, the odd one on y_j = x_{D-1-j}; box-plus is symmetric in its two
// arguments bit for bit, so with G_0 = y_0, G_i = G_{i-1} [+] y_i the even
// lane's G_i are the prefix folds F_i and the odd lane's the suffix folds
// B_{D-1-i}. Output j >= D / 2 (counted in y) is G_{j-1} [+] P_{D-2-j}, P the
// neighbour's folds, and the last one G_{D-2}. y[0 .. D / 2): this lane's
// inputs; out[i]: output D / 2 + i. 3 (D - 2) / 2 box-plus steps per lane and
// D - 2 stages of one or two, against stages of two or four with one lane per
// check.
__device__ __forceinline__ float pair_swap(float x) {  // the neighbour's value (lanes 2i and 2i + 1)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));
}
template <int D, bool FAR, int S>
__device__ __forceinline__ void boxplus_pair_stage(const float* y, float* G, float* out) {
  if constexpr (S <= D - 2) {
    if constexpr (S < D / 2) {
      boxplus<FAR, 1>(&G[S - 1], &y[S], &G[S]);
    } else {
      const float a[2] = {G[S - 1], G[S - 1]}, b[2] = {y[S], pair_swap(G[D - 2 - S])};
      float o[2];
      boxplus<FAR, 2>(a, b, o);
      G[S] = o[0];
      out[S - D / 2] = o[1];
    }
    boxplus_pair_stage<D, FAR, S + 1>(y, G, out);
  }
}
template <int D, bool FAR>
__device__ __forceinline__ void boxplus_pair_folds(const float* y, float* out) {
  float G[D];
  G[0] = y[0] + 0.0f;
  boxplus_pair_stage<D, FAR, 1>(y, G, out);
  out[D / 2 - 1] = G[D - 2];
}
template <int D>
__device__ __forceinline__ void boxplus_pair(const float* half, float* out) {
  static_assert(D == 4 || D == 6, "even degrees with a box-plus step");
  float y[D];
  float mn = fabsf(half[0]);
#pragma unroll
  for (int j = 0; j < D / 2; ++j) {
    y[j] = half[j];
    y[D - 1 - j] = pair_swap(half[j]);
    mn = fminf(mn, fabsf(half[j]));
  }
  if (__builtin_amdgcn_ballot_w64(mn < box_far_bound<D>()) == 0ull)
    boxplus_pair_folds<D, true>(y, out);
  else
    boxplus_pair_folds<D, false>(y, out);
}

// The folds of a check of degree deg in a variant with DC slots (REG: deg =
// DC). Inputs x[0 .. deg). Wavefronts whose checks all have degree DC, or
// all DC - 1, take the unrolled folds of that degree (the two degrees of the
// spacetime window codes); mixed ones the folds with a condition per slot.
template <int DC, bool REG, bool LEAN = false>
__device__ __forceinline__ void boxplus_others(const float* x, int32_t deg, float* acc) {
  if constexpr (REG) {
    boxplus_all<DC, LEAN>(x, acc);
    return;
  }
  if constexpr (DC <= 6 && DC > 2) {
    if (__builtin_amdgcn_ballot_w64(deg != DC) == 0ull) {
      boxplus_all<DC>(x, acc);
      return;
    }
    if (__builtin_amdgcn_ballot_w64(deg != DC - 1) == 0ull) {
      boxplus_all<DC - 1>(x, acc);
      return;
    }
  }
  float F[DC], B[DC];
  F[0] = x[0] + 0.0f;
#pragma unroll
  for (int k = 1; k < DC; ++k) F[k] = (k < deg) ? boxplus1(F[k - 1], x[k]) : F[k - 1];
  B[DC - 1] = (DC - 1 < deg) ? x[DC - 1] + 0.0f : __builtin_inff();
#pragma unroll
  for (int k = DC - 2; k >= 0; --k)
    B[k] = (k >= deg) ? __builtin_inff() : (k == deg - 1 ? x[k] + 0.0f : boxplus1(x[k], B[k + 1]));
#pragma unroll
  for (int j = 0; j < DC; ++j) {
    if (j >= deg) continue;
    if (j == 0)
      acc[j] = (deg >= 2) ? B[1] : __builtin_inff();
    else if (j == deg - 1)
      acc[j] = F[j - 1];
    else
      acc[j] = boxplus1(F[j - 1], B[j + 1]);
  }
}

}  // namespace laim

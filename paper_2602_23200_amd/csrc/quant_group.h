// Group arithmetic of the quantiser and what its launches share (index arithmetic, window copies).
// Every translation unit that includes this is compiled with -ffp-contract=off: the integer codes
// and the symmetric/asymmetric flag depend on every fp32 rounding, so each multiply, add, subtract
// and divide below is a separate IEEE operation (Section "Quantization Scheme", Eq. asym_quant;
// Figure "hybrid"); where a fused one is written, the comment says why it rounds alike.
#pragma once

#include "innerq_dev.h"

namespace innerq {
namespace {

__device__ inline float h2f(__half h) { return __half2float(h); }

// One quantisation group of G values.
//   asymmetric (Eq. asym_quant):  Z = min, S = (max - Z) / (2^b - 1), code = clip(rint((x - Z) / S), 0, 2^b-1)
//   symmetric:                    S = max|x| / den, code = clip(rint(x / S), -2^(b-1), 2^(b-1)-1)
//   hybrid (Figure "hybrid"):     both; L1 reconstruction errors summed in index order; asymmetric
//                                 only if its error is strictly smaller
// The scale is rounded to fp16 (its stored precision) before the codes are formed.
// Stored field: code (asymmetric) or code + 2^(b-1) (symmetric); scale sign bit = asymmetric.
// The correctly rounded fp32 quotient num / S, given r = fl(1 / S) correctly rounded (one IEEE
// division per group instead of one per element): q0 = fl(num * r) is within one ulp, the
// remainder num - S * q0 is exact in the fused multiply-add, and q0 + rem * r then rounds to
// the nearest fp32 to num / S (Markstein's division step; no underflow at these magnitudes:
// num is a multiple of 2^-24 below 2^17, S an fp16 value).  Callers pass r = 0 for S == 0.
__device__ inline float code_quotient(float num, float S, float r) {
  const float q0 = num * r;
  const float rem = __builtin_fmaf(-S, q0, num);
  return __builtin_fmaf(rem, r, q0);
}

// 1 / S for code_quotient, 0 for S == 0: every quotient of such a group is then exactly 0, which
// is the code the formula assigns when the scale is 0.
__device__ inline float group_reciprocal(float S) { return S == 0.f ? 0.f : 1.0f / S; }

// The same number in half the instructions, for an fp16 value S: one Newton step from the instruction's approximation (one
// ulp) rounds correctly for each of the 1024 significands that S can have; an infinite or NaN S is set right at the end.
__device__ inline float fp16_reciprocal(float S) {
  const float r = __builtin_amdgcn_rcpf(S);
  const float q = __builtin_fmaf(__builtin_fmaf(-S, r, 1.0f), r, r);
  return S == 0.f ? 0.f : __builtin_amdgcn_div_fixupf(q, S, 1.0f);
}
// The correctly rounded x / d for a denominator d of the scales (1, 3, 7 or 15; r = fl(1 / d)): the division step of
// code_quotient, an infinite or NaN x set right at the end.
__device__ inline float scale_quotient(float x, float d, float r) {
  return __builtin_amdgcn_div_fixupf(code_quotient(x, d, r), d, x);
}

// ---- a group in one lane: the form of prompts and chunks, and of per-channel groups but for those of short calls.  Long prompts are bound by memory, at
// the rate of a copy (8 x 8 heads x 32k tokens, 2 bits: 1.24 GB in 250 us), with the vector units busy for three quarters of it.
//
// It uses these facts, so that codes, flags and scales keep every bit:
//   * rint(fl(num / S)) is the exact quotient rounded to nearest-even.  A tie k + 1/2 of the quotient is
//     num = T = S (k + 1/2), a number of at most 16 bits and so an fp32 number; any other num is at least one
//     fp32 step from T, which leaves num / S further from k + 1/2 than half an fp32 step there.
//     The quotient may therefore be formed with any error below 2^-41 of itself before its one rounding:
//     fl(num * r_hi + fl(num * r_lo)) with r_hi + r_lo = 1 / S (1 + 2^-47), two operations where the
//     correctly rounded quotient takes three;
//   * S * code is exact (11 bits by at most 4), so the reconstruction and the symmetric difference are one
//     fused operation each;
//   * fields are collected as c * 2^(b i) in fp32, up to 16 bits at a time, exact.
// Values stay packed as they were loaded: every use is a mixed-precision multiply-add that reads its half.
// A code cannot leave its range unless the scale is an fp16 denormal (whose rounding is coarse) or the
// symmetric denominator is the literal one: wavefronts with such a group run the form that clamps.
// The competition of the two variants is decided on a shorter error sum where its rounding cannot matter (bulk_codes; in long prompts).
// Instructions per element of a 2-bit hybrid group, minimum and maximum included: 12 (14 with the oracle's own sum, 28 with
// divisions and conversions); 14 and 10 more a group for its scales and their reciprocals (45 with divisions).  Appends of 8 x 8
// heads x 32k tokens: 2 bits 259 us -> 250, 4 bits 287 -> 277, G = 64 256 -> 244.

// One value of a group: a half of a register.
struct HalfRef { uint32_t w; bool hi; };
__device__ __forceinline__ float value_of(HalfRef x) {
  return h2f(__ushort_as_half((unsigned short)(x.hi ? x.w >> 16 : x.w & 0xffffu)));
}
// 1 in a register that the compiler knows nothing about: x * 1 + c is then one mixed-precision instruction on the
// packed x instead of a conversion and an addition.
__device__ __forceinline__ float opaque_one() {
  float one = 1.0f;
  asm volatile("" : "+v"(one));      // (volatile: a 1 for each form of the loop, so that nothing of it is hoisted out of the choice)
  return one;
}
// x - b, x * r + c, x - S * c, fl(x * r), each rounded once (x an fp16 value).  The last one adds -0, so that a zero
// keeps the product's sign.
__device__ __forceinline__ float half_minus(HalfRef x, float b, float one) { return __builtin_fmaf(value_of(x), one, -b); }
__device__ __forceinline__ float half_times_plus(HalfRef x, float r, float c) { return __builtin_fmaf(value_of(x), r, c); }
__device__ __forceinline__ float half_minus_product(HalfRef x, float S, float c) { return __builtin_fmaf(-S, c, value_of(x)); }
__device__ __forceinline__ float half_times(HalfRef x, float r) {
  float d;
  if (x.hi) asm("v_fma_mix_f32 %0, %1, %2, neg(0) op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(x.w), "v"(r));
  else asm("v_fma_mix_f32 %0, %1, %2, neg(0) op_sel_hi:[1,0,0]" : "=v"(d) : "v"(x.w), "v"(r));
  return d;
}

// The two pieces of 1 / S (0 for S == 0: every code is then 0).
struct Reciprocal { float hi, lo; };
__device__ inline Reciprocal split_reciprocal(float S) {
  Reciprocal r;
  r.hi = fp16_reciprocal(S);
  r.lo = __builtin_fmaf(-S, r.hi, S == 0.f ? 0.f : 1.0f) * r.hi;    // 1 - S r_hi is exact
  return r;
}
__device__ inline float exact_code(float num, const Reciprocal& r) {
  return rintf(__builtin_fmaf(num, r.hi, num * r.lo));
}
__device__ inline float exact_code(HalfRef x, const Reciprocal& r) {
  return rintf(half_times_plus(x, r.hi, half_times(x, r.lo)));
}

// Fields of a group collected into 32-bit words; 3-bit fields as a plane of 2-bit low parts followed by a
// plane of high bits.  add(i, c): the field of element i is c + BIAS, an integer as fp32; i ascending and a
// constant after unrolling.
template <int G, int BITS, int BIAS>
struct FieldPacker {
  static constexpr int LB = BITS == 3 ? 2 : BITS;        // width in the (low) plane
  static constexpr int P = 16 / LB;                      // fields per 16 bits
  float low[G / P], high[BITS == 3 ? G / 16 : 1];
  __device__ __forceinline__ void start() {
    float all = 0.f;
#pragma unroll
    for (int i = 0; i < P; ++i) all += (float)(BIAS << (LB * i));
#pragma unroll
    for (int i = 0; i < G / P; ++i) low[i] = all;
    if constexpr (BITS == 3) {
#pragma unroll
      for (int i = 0; i < G / 16; ++i) high[i] = 0.f;
    }
  }
  __device__ __forceinline__ void add(int i, float c) {
    low[i / P] = __builtin_fmaf(c, (float)(1 << (LB * (i % P))), low[i / P]);
    if constexpr (BITS == 3) {
      const float h = __builtin_amdgcn_fmed3f(c + (float)(BIAS - 3), 0.f, 1.f);      // field >= 4
      low[i / P] = __builtin_fmaf(h, (float)(-4 * (1 << (LB * (i % P)))), low[i / P]);
      high[i / 16] = __builtin_fmaf(h, (float)(1 << (i % 16)), high[i / 16]);
    }
  }
  __device__ __forceinline__ uint32_t word(int w) const {
    constexpr int WL = G * LB / 32;
    const float lo = w < WL ? low[2 * w] : high[2 * (w - WL)], hi = w < WL ? low[2 * w + 1] : high[2 * (w - WL) + 1];
    return (uint32_t)lo | ((uint32_t)hi << 16);
  }
};

// Symmetric 2-bit codes with S = max |x| (denominator 1): -1, 0, 1 with one tie, |x| = S / 2, which goes to 0.
// The reciprocal is taken 2^-20 too small: the tie then falls below 1/2 and the next fp16 number above it
// (2^-11 away) does not.  Adding 1.5 * 2^23 leaves the code in the low bits.
template <int G>
struct TernaryPacker {
  uint32_t w[G / 16];
  __device__ __forceinline__ void start() {
    uint32_t off = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) off += (2u - 0x4B400000u) << (2 * i);    // field = code + 2; 0x4B400000: the bits of 1.5 * 2^23
#pragma unroll
    for (int i = 0; i < G / 16; ++i) w[i] = off;
  }
  // t: x * r + 1.5 * 2^23.  (one v_lshl_add_u32; the compiler makes it one and a half)
  __device__ __forceinline__ void add(int i, float t) {
    asm("v_lshl_add_u32 %0, %1, %2, %0" : "+v"(w[i / 16]) : "v"(t), "n"(2 * (i % 16)));
  }
  __device__ __forceinline__ uint32_t word(int i) const { return w[i]; }
};

// Distances |x - S code| of symmetric 2-bit groups as packed fp16 pairs: min(|x|, S - |x|) with S = max |x|.  Exact: S - |x| is where it
// is the smaller one.  The error sum takes them with one mixed-precision addition each.
__device__ __forceinline__ uint32_t ternary_distances(uint32_t x, uint32_t scales) {
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  const f16x2 a = __builtin_bit_cast(f16x2, x & 0x7fff7fffu), b = __builtin_bit_cast(f16x2, scales) - a;
  uint32_t d;                                            // (the builtin makes the minimum of a number and itself first)
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
struct NoDistances {};                                   // (the sum forms its own)

// CLAMP: codes are clamped, and `mode` (else: MODE) is what chooses between the two variants.
// FAST, where both variants compete and no code is clamped: the asymmetric differences are taken as (x - mn) - Sa code, one operation
// less than x - (Sa code + mn).  Their sum differs in its last bits, and is only compared with the other one: the result says
// whether that could change the answer (the codes of both variants are right in any case).  most: the largest magnitude.
template <int G, int BITS, int MODE, bool CLAMP, bool FAST, typename X, typename Dist>
__device__ __forceinline__ bool bulk_codes(X x, Dist dist, float mn, float most, __half Sa, __half Ss, int mode,
                                           uint32_t (&words)[G * BITS / 32], __half& scale, __half& zero) {
  constexpr bool ASYM = MODE != INNERQ_SYM, SYM = MODE != INNERQ_ASYM, BOTH = ASYM && SYM;
  constexpr bool TERNARY = BITS == 2 && !CLAMP, SHORT = BOTH && !CLAMP && FAST;
  constexpr int HALF = 1 << (BITS - 1), QMAX = (1 << BITS) - 1;
  const float Saf = h2f(Sa), Ssf = h2f(Ss);
  Reciprocal ra = {0.f, 0.f}, rs = {0.f, 0.f};
  if constexpr (ASYM) ra = split_reciprocal(Saf);
  if constexpr (SYM) rs = split_reciprocal(Ssf);
  const float r_tern = rs.hi * (1.0f - 0x1p-20f);
  FieldPacker<G, BITS, 0> pa;
  FieldPacker<G, BITS, HALF> ps;
  TernaryPacker<G> pt;
  if constexpr (ASYM) pa.start();
  if constexpr (SYM) { if constexpr (TERNARY) pt.start(); else ps.start(); }
  float ea = 0.f, es = 0.f;
  const float one = opaque_one();
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const HalfRef v = x(i);
    if constexpr (ASYM) {
      const float num = half_minus(v, mn, one);
      float c = exact_code(num, ra);
      if constexpr (CLAMP) c = __builtin_amdgcn_fmed3f(c, 0.f, (float)QMAX);
      pa.add(i, c);
      if constexpr (SHORT) ea = ea + fabsf(__builtin_fmaf(-Saf, c, num));
      else if constexpr (BOTH) ea = ea + fabsf(half_minus(v, __builtin_fmaf(Saf, c, mn), one));
    }
    if constexpr (SYM) {
      float c;
      if constexpr (TERNARY) {
        const float t = half_times_plus(v, r_tern, 12582912.0f);
        pt.add(i, t);
        if constexpr (BOTH && !__is_same(Dist, NoDistances)) {
          es = __builtin_fmaf(value_of(dist(i)), one, es);
          continue;
        }
        c = t - 12582912.0f;
      } else {
        c = exact_code(v, rs);
        if constexpr (CLAMP) c = __builtin_amdgcn_fmed3f(c, (float)(-HALF), (float)(HALF - 1));
        ps.add(i, c);
      }
      if constexpr (BOTH) es = es + fabsf(half_minus_product(v, Ssf, c));
    }
  }
  // (one condition, bitwise: entered from two tests, the arm "asymmetric" may lose the negation of its scale; see quantize_group_lanes)
  const bool asym = CLAMP ? (mode == INNERQ_ASYM) | ((mode == INNERQ_HYBRID) & (ea < es)) : BOTH ? ea < es : ASYM;
#pragma unroll
  for (int w = 0; w < G * BITS / 32; ++w) {
    uint32_t s = 0u, t = 0u;
    if constexpr (ASYM) t = pa.word(w);
    if constexpr (SYM) { if constexpr (TERNARY) s = pt.word(w); else s = ps.word(w); }
    words[w] = asym ? t : s;
  }
  scale = asym ? __hneg(Sa) : Ss;
  zero = asym ? __float2half_rn(mn) : __float2half_rn(0.f);
  if constexpr (!SHORT) return false;
  // With u = 2^-24 and M = most: x - mn, Sa code + mn and the differences round by at most (2 + 1.001 + 2 x 0.67) u M an element, and
  // the sum of each of the two ways by G u times itself.
  constexpr float u = 0x1p-24f;
  return fabsf(ea - es) < __builtin_fmaf(ea, 2.1f * G * u, most * (4.4f * G * u));
}

// The group's fields, scale and zero-point from its values x(i) and their minimum and maximum.  dist: the distances of a symmetric 2-bit
// group whose denominator is 1 (others make no use of them), or NoDistances.
// FAST: the shorter error sum, for launches that fill the chip many times over, where it gains (launch_quantize).  (One wavefront in a few hundred goes through the
// general form too, the tail of a short launch: 1 M groups of 4 bits 19.6 us and 19.8 with it, 64000 5.4 and 6.4, G = 64 8.1 and 10.2.)
template <int G, int BITS, bool FAST, typename X, typename Dist>
__device__ __forceinline__ void quantize_group_bulk(X x, Dist dist, float mn, float mx, int mode, int sym_den_literal,
                                                    uint32_t (&words)[G * BITS / 32], __half& scale, __half& zero) {
  constexpr int QMAX = (1 << BITS) - 1;
  constexpr int HALF = 1 << (BITS - 1);
  auto asym_scale = [&] { return __float2half_rn(scale_quotient(mx - mn, (float)QMAX, 1.0f / (float)QMAX)); };
  auto sym_scale = [&] {
    const float most = fmaxf(fabsf(mn), fabsf(mx));
    return __float2half_rn(sym_den_literal ? scale_quotient(most, (float)QMAX, 1.0f / (float)QMAX)
                           : HALF == 2     ? most
                                           : scale_quotient(most, (float)(HALF - 1), 1.0f / (float)(HALF - 1)));
  };
  __half Sa = asym_scale(), Ss = sym_scale();
  // a scale that is an fp16 denormal but not 0 (for 2-bit symmetric groups it is max |x| itself: exact),
  // infinite (keys that overflowed in their normalisation) or NaN (a NaN among the values)
  auto coarse = [](__half S, bool denormal) {
    const uint32_t u = __half_as_ushort(S);
    return (denormal && u != 0u && u < 0x400u) || u >= 0x7c00u;
  };
  bool clamp = (mode != INNERQ_SYM && coarse(Sa, true)) || (mode != INNERQ_ASYM && coarse(Ss, BITS != 2));
  if (sym_den_literal && mode != INNERQ_ASYM) clamp = true;
  bool redo = __builtin_amdgcn_ballot_w64(clamp) != 0;    // (wave-uniform)
  if (redo) {
    if (__builtin_amdgcn_ballot_w64(mn != mn) != 0) {
      // the packed minimum and maximum hand a NaN on; the form of eight lanes passes it over, and a token's bytes
      // do not depend on the call it came with
      mn = mx = value_of(x(0));
#pragma unroll
      for (int i = 1; i < G; ++i) {
        HalfRef v = x(i);
        asm volatile("" : "+v"(v.w));                      // (a conversion of its own: shared with the codes below it would hold a register)
        mn = fminf(mn, value_of(v));
        mx = fmaxf(mx, value_of(v));
      }
      Sa = asym_scale();
      Ss = sym_scale();
    }
  }
  if (!redo && mode == INNERQ_HYBRID)
    redo = __builtin_amdgcn_ballot_w64(bulk_codes<G, BITS, INNERQ_HYBRID, false, FAST>(x, dist, mn, fmaxf(fabsf(mn), fabsf(mx)), Sa, Ss, mode, words, scale, zero)) != 0;
  else if (!redo && mode == INNERQ_SYM) bulk_codes<G, BITS, INNERQ_SYM, false, false>(x, NoDistances{}, mn, 0.f, Sa, Ss, mode, words, scale, zero);
  else if (!redo) bulk_codes<G, BITS, INNERQ_ASYM, false, false>(x, NoDistances{}, mn, 0.f, Sa, Ss, mode, words, scale, zero);
  if (redo) {
    // The general form: clamped codes, the sums as the oracle takes them (on normal draws one wavefront in a hundred to a
    // thousand gets here).  Its inputs are opaque: whatever the compiler shared with the forms above, conversions first
    // of all, would hold registers through them (108 in the owners' kernel; 128 and 89 to 250 spilled).
    uint32_t scales = (uint32_t)__half_as_ushort(Sa) | (uint32_t)__half_as_ushort(Ss) << 16;
    asm volatile("" : "+v"(mn), "+v"(scales));
    auto again = [&](int i) {
      HalfRef v = x(i);
      asm volatile("" : "+v"(v.w));
      return v;
    };
    bulk_codes<G, BITS, INNERQ_HYBRID, true, false>(again, NoDistances{}, mn, 0.f, __ushort_as_half((unsigned short)(scales & 0xffffu)),
                                             __ushort_as_half((unsigned short)(scales >> 16)), mode, words, scale, zero);
  }
}

// Minimum / maximum of three fp16 pairs, half by half.
__device__ inline uint32_t pair_min(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ inline uint32_t pair_max(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
template <int N>
__device__ __forceinline__ void pair_range(const uint32_t (&x)[N], uint32_t& mn, uint32_t& mx) {
  mn = pair_min(x[0], x[1], x[1]);
  mx = pair_max(x[0], x[1], x[1]);
#pragma unroll
  for (int i = 2; i < N; i += 2) {
    mn = pair_min(mn, x[i], x[i + 1]);
    mx = pair_max(mx, x[i], x[i + 1]);
  }
}
__device__ inline float half_lo(uint32_t w) { return h2f(__ushort_as_half((unsigned short)(w & 0xffffu))); }
__device__ inline float half_hi(uint32_t w) { return h2f(__ushort_as_half((unsigned short)(w >> 16))); }
// A pair of keys times their normalisation factors.
// (rounded to fp32, then to fp16, as scaled_half does)
__device__ inline uint32_t scaled_pair(uint32_t w, float lo, float hi) {
  uint32_t d;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(d) : "v"(half_times(HalfRef{w, false}, lo)), "v"(half_times(HalfRef{w, true}, hi)));
  return d;
}

// Index arithmetic of one launch is 32-bit: the host refuses launches of 2^32 or more threads, token
// indices stay below 2^24 (capacity * head_dim <= 2^31), and a 64-bit division by a run-time value
// is an inlined routine of well over a hundred instructions where the 32-bit one takes about twenty.
__device__ __forceinline__ uint32_t div32(long long n, long long d) { return (uint32_t)n / (uint32_t)d; }
__device__ __forceinline__ uint32_t mod32(long long n, long long d) { return (uint32_t)n % (uint32_t)d; }

// Where the fp16 row of token t (absolute index) of sequence-head bh lives when the quantiser
// wants it: still in the recent ring if it was appended by an earlier call, else in x_new.
// (n_old: tokens cached before this call: a.n_old, or the sequence's own count.)
__device__ __forceinline__ const __half* token_row(const QuantTensorJob& j, const QuantArgs& a, long long n_old,
                                          long long bh, long long t, bool& from_new) {
  from_new = t >= n_old;
  if (from_new) return j.x_new + ((bh * a.t_new) + (t - n_old)) * kHeadDim;
  return j.ring + (bh * j.slots + mod32(t, j.slots)) * kHeadDim;
}

// Per-sequence token counts (a.n_dev: device memory, the count of every sequence before the step; Section
// "Latency", closing remark: sequences of a batch need not be equally long).  The launch is planned for
// the most any sequence can need (one key row, one value group, one window copy per sequence and head);
// each thread then takes its own sequence's state: the deferred single-token append of a cache of n0
// tokens copies token n0 into its window and quantises the rows between the states n0 + 1 and n0 + 2.
// Returns false when this sequence has nothing to quantise in this step (or is full).
__device__ __forceinline__ bool sequence_rows(const QuantArgs& a, const QuantTensorJob& j, long long bh,
                                              long long& n_old, long long& row_begin) {
  const long long n0 = a.n_dev[div32(bh, a.n_kv_heads)];
  if (n0 < 0 || n0 + 1 > a.capacity) return false;
  const long long to = n0 + 2 > a.capacity ? a.capacity : n0 + 2;
  const long long rb = quantised_rows(a.w_sink, a.w_recent, a.group, j.form, n0 + 1);
  const long long re = quantised_rows(a.w_sink, a.w_recent, a.group, j.form, to);
  n_old = n0;
  row_begin = rb;
  return re > rb;
}

// Which of the t_new new tokens (index i, absolute token n_old + i) go to a window: i < n_a to
// the sink, i >= i_b to the recent ring; the ones between were quantised by this same call.
struct CopySpan { long long n_a, i_b; };
__host__ __device__ inline CopySpan copy_span(const QuantArgs& a, long long n_old, long long ring_from) {
  long long n_a = a.w_sink - n_old;
  n_a = n_a < 0 ? 0 : (n_a > a.t_new ? a.t_new : n_a);
  long long i_b = ring_from - n_old;
  i_b = i_b < n_a ? n_a : (i_b > a.t_new ? a.t_new : i_b);
  return {n_a, i_b};
}
__host__ __device__ inline CopySpan copy_span(const QuantArgs& a, const QuantTensorJob& j) {
  return copy_span(a, a.n_old, j.ring_from);
}

// Threads the window copies of the larger of the two tensors take.
inline long long copy_threads(const QuantArgs& a) {
  long long most = 0;
  for (int w = 0; w < 2; ++w) {
    const CopySpan sp = copy_span(a, a.job[w]);
    const long long n = (long long)a.batch * a.n_kv_heads * (sp.n_a + (a.t_new - sp.i_b)) * (kHeadDim / 8);
    most = n > most ? n : most;
  }
  return most;
}

// New tokens join the fp16 windows: the sink window while it has room, otherwise the recent
// ring -- unless this same call already moved them on to the quantised store.
__device__ __forceinline__ void window_copy(const QuantArgs& a, const QuantTensorJob& j, long long idx) {
  constexpr int CPR = kHeadDim / 8;
  const long long BH = (long long)a.batch * a.n_kv_heads;
  // only the new tokens that stay in a window are visited: the first n_a (sink) and those from i_b on (ring)
  CopySpan sp = copy_span(a, j);
  const long long n_cp = sp.n_a + (a.t_new - sp.i_b);
  if (idx >= BH * n_cp * CPR) return;
  const int ch = (int)(idx % CPR);
  const long long bh = div32(idx / CPR, n_cp);
  const long long k = idx / CPR - bh * n_cp;
  long long n_old = a.n_old;
  if (a.n_dev) {
    // per-sequence count: the one new token of this sequence (the plan has n_cp = 1 for every sequence)
    const uint32_t b = div32(bh, a.n_kv_heads);
    n_old = a.n_dev[b];
    if (n_old < 0 || n_old + 1 > a.capacity) return;
    sp = copy_span(a, n_old, a.w_sink + quantised_rows(a.w_sink, a.w_recent, a.group, j.form, n_old + 1));
    // the caller's counter of this sequence moves on: one thread per sequence (a.n_dev is a copy of it)
    if (a.n_dev_out && j.is_keys && ch == 0 && mod32(bh, a.n_kv_heads) == 0) a.n_dev_out[b] = (int)(n_old + 1);
  }
  const long long i = k < sp.n_a ? k : sp.i_b + (k - sp.n_a);
  const long long t = n_old + i;
  __half* dst;
  if (t < a.w_sink) dst = j.sink + (bh * a.w_sink + t) * kHeadDim;
  else dst = j.ring + (bh * j.slots + mod32(t, j.slots)) * kHeadDim;
  uint4 raw = *reinterpret_cast<const uint4*>(j.x_new + (bh * a.t_new + i) * kHeadDim + ch * 8);
  if (j.normalise) {
    __half* h = reinterpret_cast<__half*>(&raw);
    const float* inv = a.inv_norm + mod32(bh, a.n_kv_heads) * kHeadDim + ch * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = scaled_half(h2f(h[e]), inv[e]);
  }
  *reinterpret_cast<uint4*>(dst + ch * 8) = raw;
}

// Group g of one row of the per-token form in one lane: its values at src (scaled if they are new ones and the job
// says so), its packed fields, scale and zero-point to store row lin + dr (dr apart: lin may be uniform).
template <int G, int BITS, bool FAST>
__device__ __forceinline__ void per_token_group(const QuantArgs& a, const QuantTensorJob& j, const __half* src, bool fresh,
                                                uint32_t bh, uint32_t g, long long lin, uint32_t dr) {
  constexpr int GPR = kHeadDim / G, W = G * BITS / 32;
  uint32_t x[G / 2];
#pragma unroll
  for (int i = 0; i < G / 8; ++i) {
    const uint4 raw = reinterpret_cast<const uint4*>(src)[i];
    x[4 * i] = raw.x; x[4 * i + 1] = raw.y; x[4 * i + 2] = raw.z; x[4 * i + 3] = raw.w;
  }
  if (j.normalise) {
    const float* inv = a.inv_norm + (bh % (uint32_t)a.n_kv_heads) * kHeadDim + g * G;
#pragma unroll
    for (int i = 0; i < G / 2; ++i) {
      const uint32_t y = scaled_pair(x[i], inv[2 * i], inv[2 * i + 1]);
      x[i] = fresh ? y : x[i];                           // (ring rows already are)
    }
  }
  uint32_t mn, mx;
  pair_range(x, mn, mx);
  mn = pair_min(mn, mn >> 16, mn >> 16);                 // (fminf would lose the NaN of one half and that half with it)
  mx = pair_max(mx, mx >> 16, mx >> 16);
  uint32_t words[W];
  __half s, z;
  auto value = [&](int i) { return HalfRef{x[i / 2], (i & 1) != 0}; };
  if constexpr (BITS == 2 && FAST) {
    const uint32_t less = mn ^ 0x80008000u, most = pair_max(mx, less, less) & 0xffffu, scales = most | most << 16;
    quantize_group_bulk<G, BITS, FAST>(value, [&](int i) { return HalfRef{ternary_distances(x[i / 2], scales), (i & 1) != 0}; }, half_lo(mn), half_lo(mx), j.mode,
                                 a.sym_den_literal, words, s, z);
  } else {
    quantize_group_bulk<G, BITS, FAST>(value, NoDistances{}, half_lo(mn), half_lo(mx), j.mode, a.sym_den_literal, words, s, z);
  }
  // a row is one plane of LB-bit fields over all channels (3-bit: followed by the plane of high bits)
  constexpr int LB = BITS == 3 ? 2 : BITS;
  constexpr int WL = G * LB / 32;                        // words of the (low) plane of one group
  uint32_t* rowp = reinterpret_cast<uint32_t*>(j.codes + lin * (kHeadDim * BITS / 8)) + dr * (kHeadDim * BITS / 32);
#pragma unroll
  for (int i = 0; i < WL; i += 2) *reinterpret_cast<uint2*>(rowp + g * WL + i) = uint2{words[i], words[i + 1]};
  if constexpr (BITS == 3) {
#pragma unroll
    for (int i = 0; i < G / 32; ++i) rowp[kHeadDim * 2 / 32 + g * (G / 32) + i] = words[WL + i];
  }
  (j.scales + lin * GPR)[dr * GPR + g] = s;
  if (j.zeros) (j.zeros + lin * GPR)[dr * GPR + g] = z;
}

// Job y (0: keys, 1: values) of a launch, field by field: indexing the by-value kernel argument
// with blockIdx.y makes the compiler copy the whole argument block to scratch first (so does any
// function that takes the block by reference and is not inlined: hence the forced inlining of
// quantize_rows, window_copy and token_row).
__device__ __forceinline__ QuantTensorJob pick_job(const QuantArgs& a, int y) {
  const QuantTensorJob& k = a.job[0];
  const QuantTensorJob& v = a.job[1];
  QuantTensorJob j;
  j.codes = y ? v.codes : k.codes;
  j.scales = y ? v.scales : k.scales;
  j.zeros = y ? v.zeros : k.zeros;
  j.sink = y ? v.sink : k.sink;
  j.ring = y ? v.ring : k.ring;
  j.x_new = y ? v.x_new : k.x_new;
  j.form = y ? v.form : k.form;
  j.mode = y ? v.mode : k.mode;
  j.slots = y ? v.slots : k.slots;
  j.bits = y ? v.bits : k.bits;
  j.row_begin = y ? v.row_begin : k.row_begin;
  j.row_end = y ? v.row_end : k.row_end;
  j.ring_from = y ? v.ring_from : k.ring_from;
  j.normalise = y ? v.normalise : k.normalise;
  j.is_keys = y ? 0 : 1;
  return j;
}

}  // namespace
}  // namespace innerq

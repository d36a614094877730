// The quantise work of a thread: a per-token group spread over eight lanes, a per-channel group in a lane or spread likewise,
// and the rows of one launch shared out over its threads.  Compiled without contraction (see quant_group.h); a translation unit that is
// not sets INNERQ_CONTRACTED, and the pragma below holds for this file alone.
#pragma once

#ifdef INNERQ_CONTRACTED
#pragma clang fp contract(off)
#endif
#include "quant_group.h"

namespace innerq {
namespace {

// The group quantiser spread over 8 neighbouring lanes (lane `sub` of the group holds the
// G/8 consecutive values x): the per-element divisions run in parallel, minimum / maximum are
// exact in any order, and the two error sums are still taken one element after the other in
// index order (every lane adds the whole chain from shuffled copies), so codes and flag are
// bit-identical to the form in one lane.  Returns this lane's share of the packed fields, shifted to
// its place inside its 32-bit word and OR-ed over the lanes that share that word.
template <int CTRL>
__device__ inline float lane_swap(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline uint32_t lane_swap_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// (3-bit fields: the return value is the word of the plane of 2-bit low parts, word_hi that of
// the plane of high bits, OR-ed over the lanes that share it.)
template <int G, int BITS>
__device__ inline uint32_t quantize_group_lanes(const float (&x)[G / 8], int sub, int mode, int sym_den_literal,
                                                __half& scale, __half& zero, uint32_t& word_hi) {
  constexpr int E = G / 8;
  constexpr int QMAX = (1 << BITS) - 1;
  constexpr int HALF = 1 << (BITS - 1);
  float mn = x[0], mx = x[0], am = fabsf(x[0]);
#pragma unroll
  for (int i = 1; i < E; ++i) {
    mn = fminf(mn, x[i]);
    mx = fmaxf(mx, x[i]);
    am = fmaxf(am, fabsf(x[i]));
  }
  // butterflies over the 8 lanes of the group: pairs, quads, the two quads
  mn = fminf(mn, lane_swap<0xB1>(mn)); mx = fmaxf(mx, lane_swap<0xB1>(mx)); am = fmaxf(am, lane_swap<0xB1>(am));
  mn = fminf(mn, lane_swap<0x4E>(mn)); mx = fmaxf(mx, lane_swap<0x4E>(mx)); am = fmaxf(am, lane_swap<0x4E>(am));
  mn = fminf(mn, lane_swap<0x141>(mn)); mx = fmaxf(mx, lane_swap<0x141>(mx)); am = fmaxf(am, lane_swap<0x141>(am));
  const float den = sym_den_literal ? (float)QMAX : (float)(HALF - 1);
  const __half Sa = __float2half_rn((mx - mn) / (float)QMAX);
  const __half Ss = __float2half_rn(am / den);
  const float Saf = h2f(Sa), Ssf = h2f(Ss);
  const float rSa = group_reciprocal(Saf), rSs = group_reciprocal(Ssf);
  uint32_t fa = 0u, fs = 0u, ha = 0u, hs = 0u;
  float da[E], ds[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const float ca = __builtin_amdgcn_fmed3f(rintf(code_quotient(x[i] - mn, Saf, rSa)), 0.f, (float)QMAX);
    const float cs = __builtin_amdgcn_fmed3f(rintf(code_quotient(x[i], Ssf, rSs)), (float)(-HALF), (float)(HALF - 1));
    const float ra = Saf * ca + mn;
    const float rs = Ssf * cs;
    da[i] = fabsf(x[i] - ra);
    ds[i] = fabsf(x[i] - rs);
    const uint32_t ua = (uint32_t)(int)ca, us = (uint32_t)((int)cs + HALF);
    if constexpr (BITS == 3) {
      fa |= (ua & 3u) << (i * 2);
      fs |= (us & 3u) << (i * 2);
      ha |= (ua >> 2) << i;
      hs |= (us >> 2) << i;
    } else {
      fa |= ua << (i * BITS);
      fs |= us << (i * BITS);
    }
  }
  // The two error sums in index order, as a relay over the 8 lanes: at stage s lane s of the group
  // holds the sum of all elements before its own, adds its E elements one after the other and
  // hands the result to lane s + 1 (one DPP shift).  Every lane runs every stage; only the stage
  // that matches its position produces a value that is used.  Same additions in the same order as
  // one lane summing all G values, 8 (E + 1) dependent steps instead of G cross-lane reads.
  float ra_run = 0.f, rs_run = 0.f, ea = 0.f, es = 0.f;
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    ea = ra_run;
    es = rs_run;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      ea = ea + da[i];
      es = es + ds[i];
    }
    if (st < 7) {
      ra_run = lane_swap<0x111>(ea);                     // row_shr:1: lane j takes lane j - 1's value
      rs_run = lane_swap<0x111>(es);
    }
  }
  // lane 7 of the group now holds both totals: to all 8 lanes
  const int last = ((int)(threadIdx.x & 63u) & ~7) + 7;
  ea = __shfl(ea, last);
  es = __shfl(es, last);
  // One condition, bitwise: with || and && the arm "asymmetric" is entered from two tests, and clang 22 (structurizecfg) moves the
  // negation of its scale, an instruction that costs nothing to its reckoning, in front of the first test and uses it on that edge only; lanes
  // that entered over the second one kept Ss (per-channel form, G = 64).
  const bool asym = (mode == INNERQ_ASYM) | ((mode == INNERQ_HYBRID) & (ea < es));
  scale = asym ? __hneg(Sa) : Ss;
  zero = asym ? __float2half_rn(mn) : __float2half_rn(0.f);
  constexpr int LB = BITS == 3 ? 2 : BITS;             // bits per field of the (low) plane
  constexpr int LPW = 32 / (E * LB);                   // lanes that share one 32-bit word of it
  uint32_t w = (asym ? fa : fs) << ((sub % LPW) * E * LB);
  if constexpr (LPW >= 2) w |= lane_swap_u<0xB1>(w);
  if constexpr (LPW >= 4) w |= lane_swap_u<0x4E>(w);
  word_hi = 0u;
  if constexpr (BITS == 3) {
    constexpr int LPH = 32 / E;                        // lanes per word of the high-bit plane: 8 or 4
    uint32_t h = (asym ? ha : hs) << ((sub % LPH) * E);
    h |= lane_swap_u<0xB1>(h);
    h |= lane_swap_u<0x4E>(h);
    if constexpr (LPH == 8) h |= lane_swap_u<0x141>(h);
    word_hi = h;
  }
  return w;
}

// Lane `sub` of the eight of group g of store row `row` (per-token form), whose token's values are at `token` (from_new: a new
// token's).
template <int G, int BITS>
__device__ __forceinline__ void per_token_group_lanes(const QuantArgs& a, const QuantTensorJob& j, long long bh, long long row,
                                                      int g, int sub, const __half* token, bool from_new) {
  constexpr int GPR = kHeadDim / G, E = G / 8;
  constexpr int LB = BITS == 3 ? 2 : BITS;               // bits per field of the (low) plane
  constexpr int LPW = 32 / (E * LB);
  const __half* src = token + g * G + sub * E;
  float x[E];
  if constexpr (E == 4) {
    const uint2 raw = *reinterpret_cast<const uint2*>(src);
    const __half* h = reinterpret_cast<const __half*>(&raw);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = h2f(h[e]);
  } else {
    const uint4 raw = *reinterpret_cast<const uint4*>(src);
    const __half* h = reinterpret_cast<const __half*>(&raw);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = h2f(h[e]);
  }
  if (from_new && j.normalise) {
    const float* inv = a.inv_norm + mod32(bh, a.n_kv_heads) * kHeadDim + g * G + sub * E;
#pragma unroll
    for (int i = 0; i < E; ++i) x[i] = h2f(scaled_half(x[i], inv[i]));
  }
  __half s, z;
  uint32_t word_hi;
  const uint32_t word = quantize_group_lanes<G, BITS>(x, sub, j.mode, a.sym_den_literal, s, z, word_hi);
  // a row is one plane of LB-bit fields over all channels (3-bit: followed by the plane of high bits)
  const long long lin = store_row(a.pages, a.n_kv_heads, a.capacity, bh, row);
  uint32_t* rowp = reinterpret_cast<uint32_t*>(j.codes + (lin * kHeadDim * BITS) / 8);
  if (sub % LPW == 0) rowp[g * (G * LB / 32) + sub / LPW] = word;
  if constexpr (BITS == 3) {
    constexpr int LPH = 32 / E;
    if (sub % LPH == 0) rowp[kHeadDim * 2 / 32 + g * (G / 32) + sub / LPH] = word_hi;
  }
  if (sub == 0) {
    const long long so = lin * GPR + g;
    j.scales[so] = s;
    if (j.zeros) j.zeros[so] = z;
  }
}

// Channel c of token-group tg of the store (per-channel form).  STEP: of a call with at most one new token.
template <int G, int BITS, bool STEP, bool FAST>
__device__ __forceinline__ void per_channel_group(const QuantArgs& a, const QuantTensorJob& j, long long bh, long long tg,
                                                  int c, long long n_old) {
  constexpr int W = G * BITS / 32;
  const float inv = j.normalise ? a.inv_norm[mod32(bh, a.n_kv_heads) * kHeadDim + c] : 1.f;
  const long long t0 = a.w_sink + tg * G;              // first token of the group
  const __half* fresh = j.x_new + ((bh * a.t_new) + (t0 - n_old)) * kHeadDim + c;     // (meaningful from token n_old on)
  uint32_t x[G];                                       // a value each, in the low half
  if (!STEP && t0 >= n_old) {
    // a first prompt: one base address and a fixed stride.  (Choosing between the two sources, with their 64-bit
    // addresses, for every token costs more than the group's arithmetic: a first 300 tokens of 8 heads 6.4 us against
    // 4.6 at G = 32, 9.3 against 5.8 at G = 64.)
#pragma unroll
    for (int i = 0; i < G; ++i) x[i] = __half_as_ushort(fresh[i * kHeadDim]);
    if (j.normalise) {
#pragma unroll
      for (int i = 0; i < G; ++i) x[i] = __half_as_ushort(scaled_half(h2f(__ushort_as_half((unsigned short)x[i])), inv));
    }
  } else {
    const __half* ring = j.ring + bh * j.slots * kHeadDim + c;
    uint32_t slot = mod32(t0, j.slots);
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const bool from_new = t0 + i >= n_old;
      __half v = *(from_new ? fresh + i * kHeadDim : ring + slot * kHeadDim);
      if (from_new && j.normalise) v = scaled_half(h2f(v), inv);
      x[i] = __half_as_ushort(v);
      slot = slot + 1u == (uint32_t)j.slots ? 0u : slot + 1u;
    }
  }
  uint32_t mn, mx, words[W];
  pair_range(x, mn, mx);
  __half s, z;
  quantize_group_bulk<G, BITS, FAST>([&](int i) { return HalfRef{x[i], false}; }, NoDistances{}, half_lo(mn), half_lo(mx), j.mode,
                               a.sym_den_literal, words, s, z);
  const long long go = (store_row(a.pages, a.n_kv_heads, a.capacity, bh, tg * G) / G) * kHeadDim + c;
  uint32_t* dst = reinterpret_cast<uint32_t*>(j.codes) + go * W;
#pragma unroll
  for (int i = 0; i < W; ++i) dst[i] = words[i];
  j.scales[go] = s;
  if (j.zeros) j.zeros[go] = z;
}

// Lane `sub` of the eight of channel c of token-group tg of the store (per-channel form): tokens G / 8 sub on.
template <int G, int BITS>
__device__ __forceinline__ void per_channel_group_lanes(const QuantArgs& a, const QuantTensorJob& j, long long bh, long long tg,
                                                        int c, int sub, long long n_old) {
  constexpr int E = G / 8, W = G * BITS / 32;
  constexpr int LB = BITS == 3 ? 2 : BITS, LPW = 32 / (E * LB);
  const float inv = j.normalise ? a.inv_norm[mod32(bh, a.n_kv_heads) * kHeadDim + c] : 1.f;
  const long long t0 = a.w_sink + tg * G + sub * E;    // the lane's first token
  const __half* fresh = j.x_new + ((bh * a.t_new) + (t0 - n_old)) * kHeadDim + c;     // (meaningful from token n_old on)
  const __half* ring = j.ring + bh * j.slots * kHeadDim + c;
  uint32_t slot = mod32(t0, j.slots);
  __half raw[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    raw[i] = *(t0 + i >= n_old ? fresh + i * kHeadDim : ring + slot * kHeadDim);
    slot = slot + 1u == (uint32_t)j.slots ? 0u : slot + 1u;
  }
  float x[E];
#pragma unroll
  for (int i = 0; i < E; ++i) x[i] = h2f(t0 + i >= n_old && j.normalise ? scaled_half(h2f(raw[i]), inv) : raw[i]);
  __half s, z;
  uint32_t word_hi;
  const uint32_t word = quantize_group_lanes<G, BITS>(x, sub, j.mode, a.sym_den_literal, s, z, word_hi);
  const long long go = (store_row(a.pages, a.n_kv_heads, a.capacity, bh, tg * G) / G) * kHeadDim + c;
  uint32_t* dst = reinterpret_cast<uint32_t*>(j.codes) + go * W;
  if (sub % LPW == 0) dst[sub / LPW] = word;
  if constexpr (BITS == 3) {
    constexpr int LPH = 32 / E;
    if (sub % LPH == 0) dst[G / 16 + sub / LPH] = word_hi;
  }
  if (sub == 0) {
    j.scales[go] = s;
    if (j.zeros) j.zeros[go] = z;
  }
}

// The quantise work of thread idx of tensor job j (keys and values may have different widths).  LANES: that share a
// per-token group (8, or 1).  STEP: of a call with at most one new token.  FAST: see quantize_group_bulk.
template <int G, int BITS, int LANES, bool STEP, bool FAST>
__device__ __forceinline__ void quantize_rows(const QuantArgs& a, const QuantTensorJob& j, long long idx) {
  const long long n_rows = j.row_end - j.row_begin;
  if (n_rows <= 0) return;
  const long long BH = (long long)a.batch * a.n_kv_heads;

  if (LANES == 1 && j.form == kPerToken) {
    // A lane per group, its G channels 2 G contiguous bytes; consecutive groups in consecutive lanes, over all rows and
    // sequence-heads (units of one sequence-head with scalar addresses, built first: 8 x 8 heads x 32k tokens 259 us
    // against 261 here at 2 bits, G = 32, but 325 against 277 at 4 bits, G = 64, and nothing to spread short rows over).
    constexpr int GPR = kHeadDim / G;                    // groups per row
    if (idx >= BH * n_rows * GPR) return;
    const uint32_t g = (uint32_t)idx % GPR;
    const long long bh = div32(idx / GPR, n_rows), row = j.row_begin + (idx / GPR - bh * n_rows);
    bool from_new;
    const __half* src = token_row(j, a, a.n_old, bh, a.w_sink + row, from_new) + g * G;
    per_token_group<G, BITS, FAST>(a, j, src, from_new, (uint32_t)bh, g, store_row(a.pages, a.n_kv_heads, a.capacity, bh, row), 0u);
  } else if (j.form == kPerToken) {
    // 8 lanes per group, G/8 consecutive channels each
    constexpr int GPR = kHeadDim / G;                    // groups per row
    if (idx >= BH * n_rows * GPR * 8) return;
    const int sub = (int)(idx % 8);
    const long long gi = idx / 8;
    const int g = (int)(gi % GPR);
    const long long bh = div32(gi / GPR, n_rows);
    long long n_old = a.n_old, row_begin = j.row_begin;
    if (a.n_dev && !sequence_rows(a, j, bh, n_old, row_begin)) return;
    const long long row = row_begin + (gi / GPR - bh * n_rows);
    bool from_new;
    const __half* token = token_row(j, a, n_old, bh, a.w_sink + row, from_new);
    per_token_group_lanes<G, BITS>(a, j, bh, row, g, sub, token, from_new);
  } else if (j.form == kPerChannel) {
    const long long n_groups = n_rows / G;
    if (LANES == 8 && a.channel_lanes == 8) {
      if (idx >= BH * n_groups * kHeadDim * 8) return;
      const int sub = (int)(idx % 8), c = (int)(idx / 8 % kHeadDim);
      const long long bh = div32(idx / (8 * kHeadDim), n_groups);
      long long n_old = a.n_old, row_begin = j.row_begin;
      if (a.n_dev && !sequence_rows(a, j, bh, n_old, row_begin)) return;
      per_channel_group_lanes<G, BITS>(a, j, bh, row_begin / G + (idx / (8 * kHeadDim) - bh * n_groups), c, sub, n_old);
      return;
    }
    if (idx >= BH * n_groups * kHeadDim) return;
    const int c = (int)(idx % kHeadDim);
    const long long bh = div32(idx / kHeadDim, n_groups);
    long long n_old = a.n_old, row_begin = j.row_begin;
    if (a.n_dev && !sequence_rows(a, j, bh, n_old, row_begin)) return;
    const long long tg = row_begin / G + (idx / kHeadDim - bh * n_groups);   // token-group index in the store
    per_channel_group<G, BITS, STEP, FAST>(a, j, bh, tg, c, n_old);
  } else {
    // fp16 "store": copy the rows, 8 halfs per thread
    constexpr int CPR = kHeadDim / 8;
    if (idx >= BH * n_rows * CPR) return;
    const int ch = (int)(idx % CPR);
    const long long bh = div32(idx / CPR, n_rows);
    long long n_old = a.n_old, row_begin = j.row_begin;
    if (a.n_dev && !sequence_rows(a, j, bh, n_old, row_begin)) return;
    const long long row = row_begin + (idx / CPR - bh * n_rows);
    bool from_new;
    const __half* src = token_row(j, a, n_old, bh, a.w_sink + row, from_new) + ch * 8;
    uint4 raw = *reinterpret_cast<const uint4*>(src);
    if (from_new && j.normalise) {
      __half* h = reinterpret_cast<__half*>(&raw);
      const float* inv = a.inv_norm + mod32(bh, a.n_kv_heads) * kHeadDim + ch * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = scaled_half(h2f(h[e]), inv[e]);
    }
    __half* dst = reinterpret_cast<__half*>(j.codes) + store_row(a.pages, a.n_kv_heads, a.capacity, bh, row) * kHeadDim + ch * 8;
    *reinterpret_cast<uint4*>(dst) = raw;
  }
}

// ---- the append of a decode step inside another launch, for one sequence-head and one wavefront: the key row that leaves the
// ring and both window copies.  n: tokens cached before the step; the key row between the states n + 1 and n + 2 is
// quantised.  The host: a ring of at least two tokens, so that the new one is not what leaves it.  (A value group that
// leaves, in one step of G, is a launch of its own: its code inside, four forms of G values, was most of the kernel's.)
template <int G, int KB>
__device__ __forceinline__ void append_keys_and_copies(const QuantArgs& a, long long bh, long long n, int lane) {
  constexpr int LANES = kHeadDim / G * 8;                // of the key row
  const long long to = n + 2 > a.capacity ? a.capacity : n + 2;
  const long long row = quantised_rows(a.w_sink, a.w_recent, G, kPerToken, n + 1);
  if (lane < LANES && quantised_rows(a.w_sink, a.w_recent, G, kPerToken, to) > row) {
    const QuantTensorJob j = pick_job(a, 0);
    const __half* token = j.ring + (bh * j.slots + mod32(a.w_sink + row, j.slots)) * kHeadDim;
    per_token_group_lanes<G, KB>(a, j, bh, row, lane / 8, lane % 8, token, false);
  }
  if (lane >= 32) {
    const bool values = lane >= 48;
    const int ch = lane & 15, slots = values ? a.job[1].slots : a.job[0].slots;
    __half* sink = values ? a.job[1].sink : a.job[0].sink;
    __half* ring = values ? a.job[1].ring : a.job[0].ring;
    const __half* fresh = values ? a.job[1].x_new : a.job[0].x_new;
    __half* dst = n < a.w_sink ? sink + (bh * a.w_sink + n) * kHeadDim : ring + (bh * slots + mod32(n, slots)) * kHeadDim;
    *reinterpret_cast<uint4*>(dst + ch * 8) = *reinterpret_cast<const uint4*>(fresh + bh * kHeadDim + ch * 8);
  }
}

}  // namespace
}  // namespace innerq
#ifdef INNERQ_CONTRACTED
#pragma clang fp contract(fast)
#endif

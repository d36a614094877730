// Log-sum-exp merge of the split-K partial results of one query head (Eq. att:2 over the
// concatenation of the quantised range and the windows, Figure "quantization_overall"), as a
// device function so that it can ride in more than one launch.
#pragma once

#include "innerq_dev.h"
#include "window_pass.h"

namespace innerq {

// One batch of NB partial outputs of a 64-partial chunk: every load is issued before the weights
// (which come from a separate, concurrent load) are needed.  Indices past the end re-read the last
// partial with weight zero.
template <int NB>
struct MergeBatch {
  static constexpr int D = kHeadDim;
  float2 ov[NB];
  __device__ __forceinline__ void load(const float* po, int first, int n) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int pp = k < n ? k : n - 1;
      ov[k] = *reinterpret_cast<const float2*>(po + (long long)(first + pp) * D);
    }
  }
  __device__ __forceinline__ void add(float w_l, int n, float& n0, float& n1) const {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w_l), k));
      w = k < n ? w : 0.f;
      n0 = __builtin_fmaf(w, ov[k].x, n0);          // explicit: the same rounding whatever the contraction setting
      n1 = __builtin_fmaf(w, ov[k].y, n1);
    }
  }
};

// out[b][hq][:] = sum_p w_p o_p / sum_p w_p l_p,  w_p = exp(m_p - max_p m_p).
// WAVES wavefronts of a work-group (1: any single wavefront) per query head, a lane per channel pair; the
// wavefronts take a contiguous share of the partials each and meet in LDS.  The partial outputs do not depend on the
// weights, so the loads of up to 32 of them per wavefront go out together with the loads of (m, l): one memory round
// trip for up to 32 (128 with four wavefronts) partials.
struct MergeShare { float m, den, n0, n1; };

template <int WAVES>
__device__ inline void merge_head(const AttnArgs& a, long long bhq, int wave, int lane) {
  constexpr int D = kHeadDim;
  const int n_all = a.n_valid ? a.n_valid[(uint32_t)bhq / (uint32_t)a.n_q_heads] : a.n_partials;
  const int share = (n_all + WAVES - 1) / WAVES, from = WAVES == 1 ? 0 : wave * share;
  const int P = WAVES == 1 ? n_all : (n_all - from < share ? n_all - from : share);     // (0 or less: nothing left)
  const float* ml = a.ws_ml + (bhq * a.n_partials + from) * 2;
  const float* po = a.ws_o + (bhq * a.n_partials + from) * D + 2 * lane;
  float n0 = 0.f, n1 = 0.f, den = 0.f, M = -INFINITY;
  if (WAVES == 1 || P > 0) {
    // (m, l) of partial 64 i + lane, for the first two chunks (the rest is re-read below)
    float2 mlv0 = {-INFINITY, 0.f}, mlv1 = {-INFINITY, 0.f};
    if (lane < P) mlv0 = *reinterpret_cast<const float2*>(ml + 2 * lane);
    if (64 + lane < P) mlv1 = *reinterpret_cast<const float2*>(ml + 2 * (64 + lane));
    MergeBatch<32> first;                                // partials 0 .. 31 of the first chunk
    const int n_first = P < 32 ? P : 32;
    first.load(po, 0, n_first);
    float mloc = fmaxf(mlv0.x, mlv1.x);
    for (int p = 128 + lane; p < P; p += 64) mloc = fmaxf(mloc, ml[2 * p]);
    M = window_wave_max(mloc);
    for (int base = 0; base < P; base += 64) {
      const int p_l = base + lane;
      float2 mlv = base == 0 ? mlv0 : mlv1;
      if (base >= 128 && p_l < P) mlv = *reinterpret_cast<const float2*>(ml + 2 * p_l);
      float w_l = 0.f, l_l = 0.f;
      if (p_l < P) {
        w_l = mlv.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mlv.x - M) * 1.4426950408889634f);           // an empty partial has m = -inf
        l_l = mlv.y;
      }
      float wl = w_l * l_l;
      asm("" : "+v"(wl));                               // keeps the product out of a fused add in the reduction
      den += window_wave_sum(wl);
      const int n = P - base < 64 ? P - base : 64;
      int p0 = 0;
      if (base == 0) {
        first.add(w_l, n_first, n0, n1);
        p0 = 32;
      }
      for (; p0 < n; p0 += 16) {
        MergeBatch<16> more;
        more.load(po, base + p0, n - p0 < 16 ? n - p0 : 16);
        const float w_s = __shfl(w_l, (lane + p0) & 63);
        more.add(w_s, n - p0 < 16 ? n - p0 : 16, n0, n1);
      }
    }
  }
  if constexpr (WAVES > 1) {
    __shared__ MergeShare part[WAVES][64];
    part[wave][lane] = MergeShare{M, den, n0, n1};
    __syncthreads();
    if (wave != 0) return;
    float top = M;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) top = fmaxf(top, part[w][lane].m);
    den = n0 = n1 = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const MergeShare s = part[w][lane];
      const float f = s.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s.m - top) * 1.4426950408889634f);
      den = __builtin_fmaf(f, s.den, den);
      n0 = __builtin_fmaf(f, s.n0, n0);
      n1 = __builtin_fmaf(f, s.n1, n1);
    }
  }
  const float inv = 1.0f / den;
  if (a.out_is_fp32) {
    float2 r;
    r.x = n0 * inv;
    r.y = n1 * inv;
    *reinterpret_cast<float2*>(reinterpret_cast<float*>(a.out) + bhq * D + 2 * lane) = r;
  } else {
    __half2 r = __floats2half2_rn(n0 * inv, n1 * inv);
    *reinterpret_cast<__half2*>(reinterpret_cast<__half*>(a.out) + bhq * D + 2 * lane) = r;
  }
}

// Whether a head's partials are shared by four wavefronts: where one wavefront would need a second round of loads and
// work-groups are few.  (One rule for both launches that merge, so that both give the same bits.)  Per step: 4 heads, 31
// partials 9.5 us -> 9.9, 38 10.2 -> 10.0, 512 partials 34.4 -> 17.1; 128 heads, 31 11.2 -> 11.5, 35 11.6 -> 11.2, 68 74.1 ->
// 73.1; one head alone 9.0 -> 9.4 up to 48 partials; 256 heads, 35 13.3 -> 13.7, 49 and more 20.7 -> 20.4; 512 x 36 28.0 -> 29.5
// and 1024 x 12 41.7 -> 44.7 (too many work-groups).
inline bool merge_is_shared(const AttnArgs& a) {
  const long long heads = (long long)a.batch * a.n_q_heads;
  return (a.n_partials >= 33 && heads >= 4 && heads <= 128) || (a.n_partials >= 49 && heads <= 256);
}

// ---- one launch: the work-groups of a sequence-head publish their partials and the last one to do so joins them.
//
// Every number is published as a 64-bit word together with a tag of this launch, so data and flag are one store.  A
// wavefront publishes its 64 channels of a head, waits until its stores have been performed, and then reads the words
// of all work-groups: of the wavefronts with the same channels, the one whose stores were performed last finds every
// word there, and whoever does joins them (should two find them all, both write the same bits).  Nobody waits for
// anybody.  The joiner clears the words, so a launch that is replayed from a graph with its tag finds none to begin
// with; what else the caller's workspace may hold carries the tags of no launch (31 bits, varied by lane, 66 words at a
// time).  Words are only touched by device-scope accesses (performed past the per-XCD caches), so nothing has to be
// written back or invalidated.
//
// From the barrier in front of it to the output (time stamps, 8 x 8 heads x 32k tokens): 1.1 us for the wavefronts'
// states and publishing, 0.3 until the stores are performed, 1.3 for the words, 0.5 for the sums -- against 4.7 us for a
// launch of any size behind one that fills the chip.  Arrivals counted in a word per sequence-head, the last one
// joining, take a third memory round trip and contend (32 heads x 4k tokens, attention and append 16.7 us against 14.5).
typedef unsigned long long join_word;
__device__ __forceinline__ void publish(join_word* p, float x, uint32_t tag) {
  __hip_atomic_store(p, (join_word)tag << 32 | __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ join_word look(const join_word* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void clear_word(join_word* p) { __hip_atomic_store(p, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float word_value(join_word w) { return __uint_as_float((uint32_t)w); }
__device__ __forceinline__ uint32_t word_tag(join_word w) { return (uint32_t)(w >> 32); }

// This wavefront's stores have been performed.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// w = 2^(x - top) of a partial whose level is x, both in the log2 domain (an empty partial has x = -inf).
__device__ __forceinline__ float level_weight(float x, float top) {
  return x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x - top);
}

__device__ __forceinline__ void store_output(const AttnArgs& a, long long bhq, int c, float x) {
  if (a.out_is_fp32) reinterpret_cast<float*>(a.out)[bhq * kHeadDim + c] = x;
  else reinterpret_cast<__half*>(a.out)[bhq * kHeadDim + c] = __float2half_rn(x);
}

// The words of one half (64 channels) of one head: channels [n_partials][64], then levels and sums [n_partials] each.
__device__ __forceinline__ join_word* join_words(const AttnArgs& a, long long bhq, int half) {
  return a.join + (bhq * 2 + half) * (long long)(a.n_partials * (kHeadDim / 2 + 2));
}

// Maximum / sum over the eight neighbouring lanes, in all of them.
template <int CTRL>
__device__ __forceinline__ float lane_moved(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float max_of_eight(float x) {
  x = fmaxf(x, lane_moved<0xB1>(x));
  x = fmaxf(x, lane_moved<0x4E>(x));
  return fmaxf(x, lane_moved<0x141>(x));
}
__device__ __forceinline__ float sum_of_eight(float x) {
  x += lane_moved<0xB1>(x);
  x += lane_moved<0x4E>(x);
  return x + lane_moved<0x141>(x);
}
__device__ __forceinline__ float from_lane(float x, int k) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), k));
}

// The published partials of UNITS half heads, if all are there (false for the whole wavefront else); half head u is half
// u & 1 of head u >> 1.  Up to kJoinGroups of each, so that one round of loads brings everything.
template <int UNITS>
__device__ __forceinline__ void join_published(const AttnArgs& a, long long head0, int unit, int step, int lane, int n, uint32_t tag) {
  constexpr int H = kHeadDim / 2, NB = kJoinGroups;
  static_assert(NB == 8, "a level a lane, in eight neighbouring lanes");
  const uint32_t mine = tag ^ (uint32_t)(lane << 1);
  join_word lv[UNITS], sv[UNITS], w[UNITS][NB];
#pragma unroll
  for (int i = 0; i < UNITS; ++i) {
    const int u = unit + i * step;
    const join_word* words = join_words(a, head0 + (u >> 1), u & 1);
    const join_word* levels = words + a.n_partials * H + (lane < n ? lane : n - 1);
    lv[i] = look(levels);
    sv[i] = look(levels + a.n_partials);
#pragma unroll
    for (int k = 0; k < NB; ++k) w[i][k] = look(words + (k < n ? k : n - 1) * H + lane);
  }
#pragma unroll
  for (int i = 0; i < UNITS; ++i) {
    const int u = unit + i * step;
    bool bad = lane < n && (word_tag(lv[i]) != mine || word_tag(sv[i]) != mine);
#pragma unroll
    for (int k = 0; k < NB; ++k) bad |= word_tag(w[i][k]) != mine;
    if (__builtin_amdgcn_ballot_w64(bad) != 0) continue;
    const float level = lane < n ? word_value(lv[i]) : -INFINITY;
    const float f = level_weight(level, max_of_eight(level));
    const float den = sum_of_eight(f * (lane < n ? word_value(sv[i]) : 0.f));
    float num = 0.f;
#pragma unroll
    for (int k = 0; k < NB; ++k) num = __builtin_fmaf(from_lane(f, k), word_value(w[i][k]), num);
    store_output(a, head0 + (u >> 1), (u & 1) * H + lane, num / from_lane(den, 0));
    join_word* words = join_words(a, head0 + (u >> 1), u & 1);
    for (int p = 0; p < n; ++p) clear_word(words + p * H + lane);
    if (lane < n) {
      clear_word(words + a.n_partials * H + lane);
      clear_word(words + a.n_partials * (H + 1) + lane);
    }
  }
}

// The end of a work-group of `waves` wavefronts (all of them here): their states meet in LDS (each wavefront's own
// `stride` floats of `lds`), a wavefront for every half head; then the output goes out where the sequence-head has one
// work-group, and else the partial is published and the last one joins.  Levels are in the log2 domain.
template <int NH>
__device__ __forceinline__ void join_and_store(const AttnArgs& a, const WaveState<NH>& st, float* lds, int stride, int wave,
                                               int waves, int lane, long long bh, int r, int group, int n_groups) {
  constexpr int D = kHeadDim, H = D / 2;
  static_assert(kJoinWaves == 8, "the wavefronts' levels are eight neighbouring lanes below");
  float* mine = lds + wave * stride;                     // [NH][D] outputs, then [NH][2] levels and sums
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    *reinterpret_cast<float2*>(mine + h * D + 2 * lane) = st.o[h];
    if (lane == 0) *reinterpret_cast<float2*>(mine + NH * D + 2 * h) = float2{st.m[h], st.l[h]};
  }
  __syncthreads();
  const uint32_t tag = a.join_tag;
  for (int u = wave; u < 2 * r; u += waves) {
    const int h = u >> 1, c = (u & 1) * H + lane;
    float2 ml = *reinterpret_cast<const float2*>(lds + (lane < waves ? lane : 0) * stride + NH * D + 2 * h);
    float ov[kJoinWaves], num = 0.f;
#pragma unroll
    for (int w = 0; w < kJoinWaves; ++w) ov[w] = lds[(w < waves ? w : 0) * stride + h * D + c];
    if (lane >= waves) ml = float2{-INFINITY, 0.f};
    const float top = max_of_eight(ml.x), f = level_weight(ml.x, top);
    const float den = sum_of_eight(f * ml.y);
#pragma unroll
    for (int w = 0; w < kJoinWaves; ++w) num = __builtin_fmaf(from_lane(f, w), ov[w], num);
    const long long bhq = bh * r + h;
    if (n_groups == 1) {
      store_output(a, bhq, c, num / from_lane(den, 0));
    } else {
      join_word* words = join_words(a, bhq, u & 1);
      publish(words + (long long)group * H + lane, num, tag ^ (uint32_t)(lane << 1));
      if (lane < 2)
        publish(words + (long long)a.n_partials * (H + lane) + group, lane == 0 ? top : den, tag ^ (uint32_t)(group << 1));
    }
  }
  if (n_groups == 1) return;
  stores_done();
  int u = wave;
  for (; u + waves < 2 * r; u += 2 * waves) join_published<2>(a, bh * r, u, waves, lane, n_groups, tag);
  if (u < 2 * r) join_published<1>(a, bh * r, u, waves, lane, n_groups, tag);
}

}  // namespace innerq

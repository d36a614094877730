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

}  // namespace innerq

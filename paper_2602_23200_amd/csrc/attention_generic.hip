// Attention in fp32 (any form), the short caches in one launch, and the split-K merge.
//
// attention_generic_kernel takes any grouping form and any window in fp32 (weights included).  It is the fallback for shapes
// the fused kernels do not cover, and serves the caches that hold no token quantised in both tensors yet (the first
// w_sink + w_recent + G tokens of every sequence) beyond kShortTokens tokens, in the step at which their first value group leaves, and
// for a tile with packed keys of many heads.  attention_short_kernel serves the other ones, the append of a decode step included.
// attention_merge_kernel joins all partial results by log-sum-exp: the
// quantised part and the window parts are concatenated before the softmax is
// normalised (Eq. att:1-3; Figure "quantization_overall").
#include "innerq_dev.h"
#define INNERQ_CONTRACTED
#include "quantize_rows.h"
#include "window_pass.h"
#include "merge.h"

namespace innerq {
namespace {

constexpr int D = kHeadDim;
constexpr int RT = kHeadTile;
constexpr int TILE = 64;          // tokens per inner tile

// Eight consecutive channels of one token as they are loaded: an fp16 row's 16 bytes, or the packed
// fields with the scales and zero-points that decode them.  FORM: the form of the rows that may be
// packed (kFp16: none is).
template <int FORM>
struct Octet {
  uint4 raw;            // fp16 row: 8 halves; per-token form: x = fields (3-bit: low plane), y = high plane,
                        // z = scale, w = zero-point; per-channel form: 8 fields of 4 bits in x
};
template <>
struct Octet<kPerToken> {
  uint4 raw;
  bool packed;
};
template <>
struct Octet<kPerChannel> {
  uint4 raw, s, z;      // s, z: 8 halves each
  bool packed;
};

// fp16 row of token t where the tensor keeps one (newest token, sink window, ring, fp16 store), else null.
// (This kernel also serves caches whose rows do not fit 32-bit offsets; token indices do fit.)
__device__ __forceinline__ const __half* row_of(const TensorView& tv, const AttnArgs& a, long long bh, long long t) {
  const bool is_new = tv.newest && t == a.n_tokens - 1, is_sink = t < tv.n_sink;
  const bool is_ring = t - a.w_sink >= tv.n_quant;
  const __half* base = is_new ? tv.newest + bh * D : is_sink ? tv.sink + bh * a.w_sink * D : tv.ring + bh * tv.slots * D;
  const uint32_t at = is_new ? 0u : is_sink ? (uint32_t)t : (uint32_t)t % (uint32_t)tv.slots;
  const __half* row = base + at * (uint32_t)D;
  if (is_new || is_sink || is_ring) return row;
  if (tv.form != kFp16) return nullptr;
  return reinterpret_cast<const __half*>(tv.codes) + store_row(a.pages, a.n_kv_heads, a.capacity, bh, t - a.w_sink) * D;
}

// Loads of channels 8 cb .. 8 cb + 7 of token t.  Nothing here waits for a load except the per-channel
// form, whose eight fields come from eight groups.
template <int FORM>
__device__ __forceinline__ Octet<FORM> load_octet(const TensorView& tv, const AttnArgs& a, long long bh, long long t, int cb) {
  Octet<FORM> o;
  const long long row = t - a.w_sink;                   // (meaningful beyond the sink window)
  const __half* rowp = row_of(tv, a, bh, t);
  if constexpr (FORM != kFp16) {
    o.packed = rowp == nullptr;
    if (o.packed) {
      const long long lin = store_row(a.pages, a.n_kv_heads, a.capacity, bh, row);   // (contiguous: bh * capacity + row)
      const int bits = tv.bits;
      const uint32_t G = (uint32_t)a.group;
      if constexpr (FORM == kPerToken) {
        const uint8_t* p = tv.codes + (lin * D * bits) / 8;
        const long long si = lin * (D / G) + 8 * cb / G;
        o.raw.x = bits == 4 ? *reinterpret_cast<const uint32_t*>(p + 4 * cb) : *reinterpret_cast<const unsigned short*>(p + 2 * cb);
        o.raw.y = bits == 3 ? p[D / 4 + cb] : 0u;
        o.raw.z = __half_as_ushort(tv.scales[si]);
        o.raw.w = tv.zeros ? __half_as_ushort(tv.zeros[si]) : 0u;
      } else {
        const uint32_t j = (uint32_t)row % G;              // (lin - j: the group's first row; a group never leaves its page)
        const long long si = ((lin - j) / G) * D + 8 * cb;
        const int run = G * bits / 8;                      // bytes of one channel's fields
        const uint8_t* p = tv.codes + si * run;
        uint32_t f = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint8_t* c = p + e * run;
          uint32_t u;
          if (bits == 3) u = ((c[j / 4] >> (2 * (j % 4))) & 3u) | (((c[G / 4 + j / 8] >> (j % 8)) & 1u) << 2);
          else u = (c[j * bits / 8] >> (j * bits % 8)) & ((1u << bits) - 1u);
          f |= u << (4 * e);
        }
        o.raw.x = f;
        o.s = *reinterpret_cast<const uint4*>(tv.scales + si);
        o.z = tv.zeros ? *reinterpret_cast<const uint4*>(tv.zeros + si) : uint4{0u, 0u, 0u, 0u};
      }
      return o;
    }
  }
  o.raw = *reinterpret_cast<const uint4*>(rowp + 8 * cb);
  return o;
}

__device__ inline float half_at(const uint4& v, int e) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  return h2f(__ushort_as_half((unsigned short)((e & 1) ? w[e / 2] >> 16 : w[e / 2] & 0xffffu)));
}

// Eq. hybrid_dequant: |S| * code + M * zero; a symmetric group's field is its code + 2^(b-1).  (|S| times
// a field or 2^(b-1) is exact in fp32, so the fused form rounds once, like a product and a sum do here.)
__device__ inline float decode_field(uint32_t u, float s, float z, int bits) {
  const float S = fabsf(s);
  return __builtin_fmaf(S, (float)u, (__float_as_uint(s) >> 31) ? z : -S * (float)(1 << (bits - 1)));
}
template <int FORM>
__device__ __forceinline__ void decode_octet(const Octet<FORM>& o, int bits, float (&x)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = half_at(o.raw, e);
  if constexpr (FORM == kPerToken) {
    if (o.packed) {
      const int lb = bits == 3 ? 2 : bits;               // width of the (low) plane's fields
      const float s = h2f(__ushort_as_half((unsigned short)o.raw.z)), z = h2f(__ushort_as_half((unsigned short)o.raw.w));
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[e] = decode_field(((o.raw.x >> (lb * e)) & ((1u << lb) - 1u)) | (((o.raw.y >> e) & 1u) << 2), s, z, bits);
    }
  } else if constexpr (FORM == kPerChannel) {
    if (o.packed) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = decode_field((o.raw.x >> (4 * e)) & 15u, half_at(o.s, e), half_at(o.z, e), bits);
    }
  }
}

// Sum over the 16 lanes that share a token row.
__device__ inline float row_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));
  return x;
}

// One value per row group of 16 lanes and channel of a head, o[h][e], summed over the four row groups of a
// wavefront: lanes 16 g .. 16 g + 15 get head g's eight sums.  (Each exchange takes two different values
// and leaves both of its results in use.)
__device__ __forceinline__ void add_row_groups(const float (&o)[RT][8], float (&sum)[8]) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // lower half of the wavefront: heads 0, 1; upper half: heads 2, 3
    const u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0][e]), __float_as_uint(o[2][e]), false, false);
    const u32x2 q = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[1][e]), __float_as_uint(o[3][e]), false, false);
    const float lo = __uint_as_float(p.x) + __uint_as_float(p.y), hi = __uint_as_float(q.x) + __uint_as_float(q.y);
    const u32x2 t = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    sum[e] = __uint_as_float(t.x) + __uint_as_float(t.y);
  }
}

// One work-group: up to four query heads, tiles of 64 tokens.  16 lanes share a token row (16 bytes of an
// fp16 row each, coalesced), ROWS rows a thread, and a tile's key and value loads all go out before the
// first is used.  Where a launch is one tile per work-group,
// its time is a memory round trip and the instructions of one thread, so 1024 threads take a row each
// (ROWS = 1); with several tiles per work-group, or more work-groups than compute units, 256 threads take four
// (ROWS = 4).  The kernel before this one decoded element by element: 2 x 8 heads x 165 tokens, kernel trace, 27 us (100 tokens) and 36 us
// (packed key rows among them) against 6.2 and 6.7; four rows a thread 7.6 and 8.4.  Attention call on
// longer caches (4 sequences, 8 kv heads, 4k tokens, 4-bit keys with 2-bit values): 146 us against 66.
template <int KF, int VF, int ROWS>
__global__ void __launch_bounds__(1024 / ROWS) attention_generic_kernel(AttnArgs a, long long a0, long long a1,
                                                                long long b0, long long b1, int n_chunks,
                                                                int first_slot) {
  constexpr int GROUPS = TILE / ROWS;                   // row groups of 16 lanes
  constexpr int WAVES = GROUPS / 4;
  const int tid = threadIdx.x;
  const long long bh = blockIdx.y;                      // b * Hk + hk
  const int r = a.n_q_heads / a.n_kv_heads;
  const int b = (int)blockIdx.y / a.n_kv_heads, hk = (int)blockIdx.y % a.n_kv_heads;
  const int h0 = blockIdx.z * RT;                       // first query head (within the kv head) of this pass
  const int nh = min(RT, r - h0);
  const long long na = a1 - a0, total = na + (b1 - b0);
  const long long chunk_len = (total + n_chunks - 1) / n_chunks;
  const long long v0 = (long long)blockIdx.x * chunk_len;
  const long long v1 = min(total, v0 + chunk_len);
  const int cb = tid & 15, tg = tid >> 4;               // channels 8 cb .. 8 cb + 7; token rows GROUPS k + tg of a tile
  const int wave = tid >> 6, lane = tid & 63;

  __shared__ __attribute__((aligned(16))) float s_s[RT][TILE];
  __shared__ float alpha_s[RT];
  __shared__ __attribute__((aligned(16))) float o_s[WAVES][RT][D];

  uint4 q_raw[RT];
#pragma unroll
  for (int h = 0; h < RT; ++h) {
    q_raw[h] = uint4{0u, 0u, 0u, 0u};
    if (h < nh) q_raw[h] = *reinterpret_cast<const uint4*>(a.q + ((long long)b * a.n_q_heads + hk * r + h0 + h) * D + 8 * cb);
  }
  Octet<KF> ko[ROWS];
  Octet<VF> vo[ROWS];
  auto load_rows = [&](long long base) {
    long long t[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      long long v = base + GROUPS * k + tg;
      v = v < v1 ? v : v1 - 1;                          // rows past the end re-read the last one (weight 0)
      t[k] = v < na ? a0 + v : b0 + (v - na);
      ko[k] = load_octet<KF>(a.k, a, bh, t[k], cb);
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) vo[k] = load_octet<VF>(a.v, a, bh, t[k], cb);
  };
  if (v0 < v1) load_rows(v0);

  float q[RT][8];
#pragma unroll
  for (int h = 0; h < RT; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) q[h][e] = half_at(q_raw[h], e);
  if (a.q_scale) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f = a.q_scale[hk * D + 8 * cb + e];
#pragma unroll
      for (int h = 0; h < RT; ++h) q[h][e] = h2f(scaled_half(q[h][e], f));
    }
  }

  const float sm_scale = 0.08838834764831845f;          // 1 / sqrt(128)
  float m_run = -INFINITY, l_run = 0.f;                 // running max / sum of head `wave` (wavefronts 0 .. 3)
  float o[RT][8];
#pragma unroll
  for (int h = 0; h < RT; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) o[h][e] = 0.f;

  for (long long base = v0; base < v1; base += TILE) {
    if (base != v0) load_rows(base);
    // ---- scores (Eq. att:1, scaled by 1/sqrt(d))
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      float x[8], acc[RT];
      decode_octet<KF>(ko[k], a.k.bits, x);
#pragma unroll
      for (int h = 0; h < RT; ++h) {
        acc[h] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h] = __builtin_fmaf(q[h][e], x[e], acc[h]);
        acc[h] = row_sum(acc[h]);
      }
      const float mine = cb == 0 ? acc[0] : cb == 1 ? acc[1] : cb == 2 ? acc[2] : acc[3];
      const bool valid = base + GROUPS * k + tg < v1;
      if (cb < RT) s_s[cb][GROUPS * k + tg] = valid ? mine * sm_scale : -INFINITY;
    }
    __syncthreads();
    // ---- running softmax of head `wave` (Eq. att:2), one token per lane
    if (WAVES == RT || wave < RT) {
      const float s = s_s[wave][lane];
      const float m_new = fmaxf(m_run, window_wave_max(s));
      const float p = expf(s - m_new);
      const float alpha = expf(m_run - m_new);           // 0 on the first tile (m_run = -inf)
      l_run = l_run * alpha + window_wave_sum(p);
      m_run = m_new;
      s_s[wave][lane] = p;
      if (lane == 0) alpha_s[wave] = alpha;
    }
    __syncthreads();
    // ---- weighted sum of values (Eq. att:3): the thread's channels of its token rows
    if (base != v0) {
#pragma unroll
      for (int h = 0; h < RT; ++h) {
        const float alpha = alpha_s[h];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[h][e] *= alpha;
      }
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      float x[8];
      decode_octet<VF>(vo[k], a.v.bits, x);
#pragma unroll
      for (int h = 0; h < RT; ++h) {
        const float p = s_s[h][GROUPS * k + tg];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[h][e] = __builtin_fmaf(p, x[e], o[h][e]);
      }
    }
    if (base + TILE < v1) __syncthreads();
  }

  // ---- add up the row groups and write the partial (m, l, o) of each head
  {
    float sum[8];
    add_row_groups(o, sum);
    float* dst = &o_s[wave][lane >> 4][8 * cb];
    *reinterpret_cast<float4*>(dst) = float4{sum[0], sum[1], sum[2], sum[3]};
    *reinterpret_cast<float4*>(dst + 4) = float4{sum[4], sum[5], sum[6], sum[7]};
  }
  __syncthreads();
  const int slot = first_slot + blockIdx.x;
  if (wave < nh) {                                      // wavefront = head, lane = channel pair
    float2 sum = {0.f, 0.f};
#pragma unroll
    for (int g = 0; g < WAVES; ++g) {
      const float2 x = *reinterpret_cast<const float2*>(&o_s[g][wave][2 * lane]);
      sum.x += x.x;
      sum.y += x.y;
    }
    const long long bhq = (long long)b * a.n_q_heads + hk * r + h0 + wave;
    *reinterpret_cast<float2*>(&a.ws_o[(bhq * a.n_partials + slot) * D + 2 * lane]) = sum;
    if (lane == 0) {
      a.ws_ml[(bhq * a.n_partials + slot) * 2 + 0] = m_run;
      a.ws_ml[(bhq * a.n_partials + slot) * 2 + 1] = l_run;
    }
  }
}

// q.x[2 i], q.x[2 i + 1] times the same two of an fp16 row, added to acc: two mixed-precision multiply-adds (exact products).
__device__ __forceinline__ float add_products(const uint4& q, const uint4& x, float acc) {
  const uint32_t qw[4] = {q.x, q.y, q.z, q.w}, xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc = __builtin_fmaf(half_lo(qw[i]), half_lo(xw[i]), acc);
    acc = __builtin_fmaf(half_hi(qw[i]), half_hi(xw[i]), acc);
  }
  return acc;
}

// A cache of at most kShortTokens tokens, none of them quantised in both tensors, in one launch: a work-group takes all tokens
// of a sequence-head for up to NH query heads.  16 lanes share a token row as in attention_generic_kernel; a thread has a
// row of each 64-token tile, and all its loads go out before the first is used.  The append of a decode step's token rides along as
// work-groups of its own (the last ones, a sequence-head a wavefront): a new token's ring slot is never one that the attention reads.
//
// Such a step is a memory round trip and the instructions of one work-group, so what counts is to have one launch instead of
// one for partials and one for merge and append, and few instructions a thread: products of fp16 rows are mixed-precision
// multiply-adds (exact products, no conversions), and a work-group has as few heads as the chip has room for.  GPU time of
// a step in a graph, 4-bit, before -> now: 2 x 8 heads, r = 4, 60 tokens 9.3 us -> 4.7, 128 tokens 9.3 -> 6.0, 150 (packed
// key rows among them) 10.0 -> 6.7; 32 x 8 heads, 60 9.7 -> 6.6, 150 14.5 -> 11.4; 128 x 8 heads, 60 20.0 -> 15.4, 150 40.6 -> 32.8.
// Registers: 64 a thread leave room for two work-groups a compute unit (128 x 8 heads x 128 tokens 22.5 us, 26.0 without the bound); with packed
// rows that bound spills (2 x 8 x 150 7.4 against 6.7).
template <int KF, int VF, int NH>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(KF == kFp16 && VF == kFp16 ? 8 : 4, 8))) attention_short_kernel(AttnArgs a, int r, int passes, int attention_groups, QuantArgs append) {
  constexpr int ROWS = kShortTokens / TILE, WAVES = 16, V = NH * 8;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if ((int)blockIdx.x >= attention_groups) {
    // ---- the append of the step's token, a sequence-head a wavefront: memory that the attention does not touch
    const long long bh = (long long)((int)blockIdx.x - attention_groups) * WAVES + wave;
    if (bh >= (long long)a.batch * a.n_kv_heads) return;
    const long long n = a.n_tokens - 1;
    if (a.group == 32) {
      if (a.bits == 2) append_keys_and_copies<32, 2>(append, bh, n, lane);
      else if (a.bits == 3) append_keys_and_copies<32, 3>(append, bh, n, lane);
      else append_keys_and_copies<32, 4>(append, bh, n, lane);
    } else {
      if (a.bits == 2) append_keys_and_copies<64, 2>(append, bh, n, lane);
      else if (a.bits == 3) append_keys_and_copies<64, 3>(append, bh, n, lane);
      else append_keys_and_copies<64, 4>(append, bh, n, lane);
    }
    return;
  }
  const uint32_t bh = blockIdx.x / (uint32_t)passes;
  const int h0 = (int)(blockIdx.x - bh * passes) * NH, nh = min(NH, r - h0);
  const uint32_t hk = bh % (uint32_t)a.n_kv_heads;
  const int n = (int)a.n_tokens;
  const int cb = tid & 15, tg = tid >> 4;               // channels 8 cb .. 8 cb + 7; token rows 64 k + tg

  __shared__ float s_s[NH][kShortTokens];
  __shared__ float l_s[NH];
  __shared__ __attribute__((aligned(16))) float o_s[WAVES][NH][D];

  Octet<KF> ko[ROWS];
  Octet<VF> vo[ROWS];
#pragma unroll
  for (int k = 0; k < ROWS; ++k)
    if (k == 0 || TILE * k < n) ko[k] = load_octet<KF>(a.k, a, bh, min(TILE * k + tg, n - 1), cb);     // (rows past the end: the last one, weight 0)
  uint4 q[NH];
  const long long hq = (long long)bh * r + h0;           // (batch b * n_q_heads + hk r + h0)
#pragma unroll
  for (int h = 0; h < NH; ++h) q[h] = *reinterpret_cast<const uint4*>(a.q + (hq + (h < nh ? h : 0)) * D + 8 * cb);
#pragma unroll
  for (int k = 0; k < ROWS; ++k)
    if (k == 0 || TILE * k < n) vo[k] = load_octet<VF>(a.v, a, bh, min(TILE * k + tg, n - 1), cb);
  if (a.q_scale) {
    const float4* f = reinterpret_cast<const float4*>(a.q_scale + hk * D + 8 * cb);
    const float4 f0 = f[0], f1 = f[1];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      q[h].x = scaled_pair(q[h].x, f0.x, f0.y);
      q[h].y = scaled_pair(q[h].y, f0.z, f0.w);
      q[h].z = scaled_pair(q[h].z, f1.x, f1.y);
      q[h].w = scaled_pair(q[h].w, f1.z, f1.w);
    }
  }

  // ---- scores (Eq. att:1, scaled by 1/sqrt(d))
  const float sm_scale = 0.08838834764831845f;          // 1 / sqrt(128)
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    if (k > 0 && TILE * k >= n) break;
    float acc[NH];
    bool packed = false;
    if constexpr (KF != kFp16) packed = __builtin_amdgcn_ballot_w64(ko[k].packed) != 0;    // (a wavefront's four rows: packed ones among them)
    if (packed) {
      float x[8];
      decode_octet<KF>(ko[k], a.k.bits, x);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        acc[h] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h] = __builtin_fmaf(half_at(q[h], e), x[e], acc[h]);
      }
    } else {
#pragma unroll
      for (int h = 0; h < NH; ++h) acc[h] = add_products(q[h], ko[k].raw, 0.f);
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) acc[h] = row_sum(acc[h]);
    float mine = acc[0];
#pragma unroll
    for (int h = 1; h < NH; ++h) mine = cb == h ? acc[h] : mine;
    const int t = TILE * k + tg;
    if (cb < NH) s_s[cb][t] = t < n ? mine * sm_scale : -INFINITY;
  }
  __syncthreads();
  // ---- softmax of head `wave` (Eq. att:2), a token of every tile per lane
  if (wave < NH) {
    float s[ROWS], top = -INFINITY, sum = 0.f;
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      s[k] = TILE * k < n ? s_s[wave][TILE * k + lane] : -INFINITY;
      top = fmaxf(top, s[k]);
    }
    top = window_wave_max(top);
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      if (k > 0 && TILE * k >= n) break;
      const float p = expf(s[k] - top);
      s_s[wave][TILE * k + lane] = p;
      sum += p;
    }
    sum = window_wave_sum(sum);
    if (lane == 0) l_s[wave] = sum;
  }
  __syncthreads();
  // ---- weighted sum of values (Eq. att:3): the thread's channels of its token rows
  float o[V];
#pragma unroll
  for (int i = 0; i < V; ++i) o[i] = 0.f;
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    if (k > 0 && TILE * k >= n) break;
    float x[8];
    decode_octet<VF>(vo[k], a.v.bits, x);
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const float p = s_s[h][TILE * k + tg];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[8 * h + e] = __builtin_fmaf(p, x[e], o[8 * h + e]);
    }
  }
  // ---- the wavefront's four rows, each keeping a quarter of the (head, channel) sums; then the wavefronts
  {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    float half[V / 2], quarter[V / 4];
#pragma unroll
    for (int i = 0; i < V / 2; ++i) {
      const u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[i]), __float_as_uint(o[V / 2 + i]), false, false);
      half[i] = __uint_as_float(p.x) + __uint_as_float(p.y);
    }
#pragma unroll
    for (int i = 0; i < V / 4; ++i) {
      const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(half[i]), __float_as_uint(half[V / 4 + i]), false, false);
      quarter[i] = __uint_as_float(p.x) + __uint_as_float(p.y);
    }
    const int at = (lane >> 4) * (V / 4);                // of the V sums of channel block cb: head at / 8, channels at % 8 on
    float* dst = &o_s[wave][at / 8][8 * cb + at % 8];
#pragma unroll
    for (int i = 0; i < V / 4; i += 2) *reinterpret_cast<float2*>(dst + i) = float2{quarter[i], quarter[i + 1]};
  }
  __syncthreads();
  if (wave < nh) {                                      // wavefront = head, lane = channel pair
    float2 sum = {0.f, 0.f};
#pragma unroll
    for (int g = 0; g < WAVES; ++g) {
      const float2 x = *reinterpret_cast<const float2*>(&o_s[g][wave][2 * lane]);
      sum.x += x.x;
      sum.y += x.y;
    }
    const float inv = 1.0f / l_s[wave];
    const long long at = (hq + wave) * D + 2 * lane;
    if (a.out_is_fp32) *reinterpret_cast<float2*>(reinterpret_cast<float*>(a.out) + at) = float2{sum.x * inv, sum.y * inv};
    else *reinterpret_cast<__half2*>(reinterpret_cast<__half*>(a.out) + at) = __floats2half2_rn(sum.x * inv, sum.y * inv);
  }
}

template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) attention_merge_kernel(AttnArgs a) {
  merge_head<WAVES>(a, blockIdx.x, threadIdx.x >> 6, threadIdx.x & 63);
}

}  // namespace

hipError_t launch_attention_generic(const AttnArgs& a, long long a0, long long a1, long long b0, long long b1,
                                    int n_chunks, int first_slot, hipStream_t stream) {
  const int r = a.n_q_heads / a.n_kv_heads;
  dim3 grid((unsigned)n_chunks, (unsigned)(a.batch * a.n_kv_heads), (unsigned)((r + RT - 1) / RT));
  // Which rows of the two ranges a tensor keeps packed: none unless it has quantised rows inside them.
  // (A kernel that can meet a form carries its decode: 12.3 us instead of 8.7 on 16 x 165 tokens.)
  auto packed_form = [&](const TensorView& tv) -> int {
    const long long q0 = a.w_sink, q1 = a.w_sink + tv.n_quant;
    const bool some = tv.form != kFp16 && ((a0 < q1 && a1 > q0 && a1 > a0) || (b0 < q1 && b1 > q0 && b1 > b0));
    return some ? tv.form : (int)kFp16;
  };
  const int kf = packed_form(a.k), vf = packed_form(a.v);
  const long long tokens = (a1 - a0) + (b1 - b0);
  // A row a thread while every work-group has a compute unit to itself (16 x 8 heads, 70 tokens, 256 work-groups: step
  // 9.3 us against 9.9); beyond, work-groups of 1024 threads wait for one another (129 tokens, 384 of them: 13.3 against
  // 11.1; 256 x 8 heads, one token: 35.8 against 20.7).
  const bool one_row_each =
      (tokens + n_chunks - 1) / n_chunks <= TILE && (long long)grid.x * grid.y * grid.z <= (long long)compute_units();
  auto go = [&](auto one_row, auto four_rows) {
    if (one_row_each) one_row<<<grid, 1024, 0, stream>>>(a, a0, a1, b0, b1, n_chunks, first_slot);
    else four_rows<<<grid, 256, 0, stream>>>(a, a0, a1, b0, b1, n_chunks, first_slot);
    return hipGetLastError();
  };
  if (kf == kFp16) {
    if (vf == kFp16) return go(attention_generic_kernel<kFp16, kFp16, 1>, attention_generic_kernel<kFp16, kFp16, 4>);
    if (vf == kPerToken) return go(attention_generic_kernel<kFp16, kPerToken, 1>, attention_generic_kernel<kFp16, kPerToken, 4>);
    return go(attention_generic_kernel<kFp16, kPerChannel, 1>, attention_generic_kernel<kFp16, kPerChannel, 4>);
  }
  if (kf == kPerToken) {
    if (vf == kFp16) return go(attention_generic_kernel<kPerToken, kFp16, 1>, attention_generic_kernel<kPerToken, kFp16, 4>);
    return go(attention_generic_kernel<kPerToken, kPerChannel, 1>, attention_generic_kernel<kPerToken, kPerChannel, 4>);
  }
  if (vf == kFp16) return go(attention_generic_kernel<kPerChannel, kFp16, 1>, attention_generic_kernel<kPerChannel, kFp16, 4>);
  return go(attention_generic_kernel<kPerChannel, kPerToken, 1>, attention_generic_kernel<kPerChannel, kPerToken, 4>);
}

hipError_t launch_attention_short(const AttnArgs& a, const QuantArgs* append, hipStream_t stream) {
  const int r = a.n_q_heads / a.n_kv_heads, bh = a.batch * a.n_kv_heads;
  const bool kp = a.k.form != kFp16 && a.k.n_quant > 0, vp = a.v.form != kFp16 && a.v.n_quant > 0;
  if ((kp && vp) || (kp && a.k.form != kPerToken) || (vp && a.v.form != kPerToken)) return hipErrorInvalidValue;
  // One query head a work-group while every work-group, the append's among them, has a compute unit to itself, else two, else four
  // (us a step, one, two and four heads each: 2 x 8 kv heads, r = 4, 128 tokens 6.0, 6.5, 7.7; 8 x 8, 260, 132 and 68 work-groups, 150
  // tokens 9.6, 7.5, 8.5; 32 x 8, 128 tokens 15.4, 9.5, 8.6).  Heads that are there: one of one stays one (128 x 8 kv heads, r = 1 12.4, 18.8 in four).
  const int append_groups = append ? (bh + 15) / 16 : 0;
  int heads_each = 1;
  while (heads_each < RT && heads_each < r && (long long)bh * ((r + heads_each - 1) / heads_each) + append_groups > compute_units()) heads_each *= 2;
  const int passes = (r + heads_each - 1) / heads_each, groups = bh * passes;
  const dim3 grid((unsigned)(groups + append_groups));
  auto go = [&](auto kernel) {
    kernel<<<grid, 1024, 0, stream>>>(a, r, passes, groups, append ? *append : QuantArgs{});
    return hipGetLastError();
  };
  auto heads = [&](auto k1, auto k2, auto k4) { return heads_each == 1 ? go(k1) : heads_each == 2 ? go(k2) : go(k4); };
  if (kp) return heads(attention_short_kernel<kPerToken, kFp16, 1>, attention_short_kernel<kPerToken, kFp16, 2>, attention_short_kernel<kPerToken, kFp16, 4>);
  if (vp) return heads(attention_short_kernel<kFp16, kPerToken, 1>, attention_short_kernel<kFp16, kPerToken, 2>, attention_short_kernel<kFp16, kPerToken, 4>);
  return heads(attention_short_kernel<kFp16, kFp16, 1>, attention_short_kernel<kFp16, kFp16, 2>, attention_short_kernel<kFp16, kFp16, 4>);
}

hipError_t launch_attention_merge(const AttnArgs& a, hipStream_t stream) {
  const unsigned heads = (unsigned)(a.batch * a.n_q_heads);
  if (merge_is_shared(a)) attention_merge_kernel<4><<<heads, 256, 0, stream>>>(a);
  else attention_merge_kernel<1><<<heads, 64, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace innerq

// Bulk appends (a prompt or a chunk of one): quantise, pack and copy into the windows in one launch.
//
// What bounds it: vector instructions, with memory close behind (2-bit hybrid groups: 14 instructions and 2.4
// bytes moved per element).  So everything that is the same for a wavefront is kept out of the lanes:
//   * a wavefront of the per-token form takes 64 consecutive groups of one sequence-head, one a lane: its G
//     channels are 2 G contiguous bytes, and the 64 lanes' loads and packed stores are contiguous too;
//   * a wavefront of the per-channel form takes one group of G tokens, a lane a pair of channels: a token's row
//     is one coalesced 256-byte load.
// One wavefront, one such unit; four wavefronts per SIMD hide the loads.  (Resident wavefronts that walk over
// the units with the next unit's loads in flight were built first: 317 us against 301 for one unit each, with
// the same arithmetic, on 8 x 8 heads x 32k tokens: copies and spills cost more than the latency they hid.)
// Tokens that leave the recent ring are read by the same work-group that afterwards writes the new tokens
// into it, one work-group per sequence-head, tensor and slice of G channels, so a call needs no second launch.
//
// Measured against one group a lane in a kernel of all forms (quotients in three operations, values converted
// first, copies in a second launch): 8 x 8 heads x 32k tokens, 2-bit hybrid, G = 32, append 364 us -> 262, with key
// factors 383 -> 278; G = 64, 16k tokens 191 -> 142; 3-bit, 16k tokens 243 -> 182; a 512-token chunk onto 500 tokens of
// 8 heads 10.2 -> 7.7.
#include "innerq_dev.h"
#include "quant_group.h"

#ifndef INNERQ_BULK_GROUP
#define INNERQ_BULK_GROUP 32
#endif

namespace innerq {
namespace {

constexpr int G = INNERQ_BULK_GROUP;
constexpr int D = kHeadDim;

// ---- per-token form ------------------------------------------------------------------------
// 64 groups: rows row0 .. row0 + 64 / GPR of sequence-head bh, or (RING) rows row0 .. row0 + 63 of one channel
// slice.  Rows from row_end on are not there: their lanes repeat the last one, store included.
template <int BITS, bool RING>
__device__ __forceinline__ void per_token_unit(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t row0,
                                               uint32_t row_end, uint32_t slice) {
  constexpr uint32_t GPR = D / G;                        // groups per row
  constexpr int W = G * BITS / 32;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t g = RING ? slice : lane % GPR;
  uint32_t r = RING ? lane : lane / GPR;                 // row within the unit
  r = row0 + r < row_end ? r : row_end - 1u - row0;
  const __half* base = j.x_new + ((long long)bh * a.t_new + ((long long)a.w_sink + row0 - a.n_old)) * D;   // (uniform)
  bool fresh = true;                                     // not from the ring
  const __half* src = base + (r * D + g * G);
  if (RING) {
    const long long t = (long long)a.w_sink + row0 + r;
    fresh = t >= a.n_old;
    const __half* old = j.ring + ((long long)bh * j.slots + (uint32_t)t % (uint32_t)j.slots) * D + g * G;
    src = fresh ? src : old;
  }
  uint32_t x[G / 2];
#pragma unroll
  for (int i = 0; i < G / 8; ++i) {
    const uint4 raw = reinterpret_cast<const uint4*>(src)[i];
    x[4 * i] = raw.x; x[4 * i + 1] = raw.y; x[4 * i + 2] = raw.z; x[4 * i + 3] = raw.w;
  }
  if (j.normalise) {
    const float* inv = a.inv_norm + (bh % (uint32_t)a.n_kv_heads) * D + g * G;
#pragma unroll
    for (int i = 0; i < G / 2; ++i) {
      const uint32_t y = scaled_pair(x[i], inv[2 * i], inv[2 * i + 1]);
      x[i] = !RING || fresh ? y : x[i];                  // (ring rows already are)
    }
  }
  uint32_t mn, mx;
  pair_range(x, mn, mx);
  uint32_t words[W];
  __half s, z;
  mn = pair_min(mn, mn >> 16, mn >> 16);                 // (fminf would lose the NaN of one half and that half with it)
  mx = pair_max(mx, mx >> 16, mx >> 16);
  quantize_group_bulk<G, BITS>([&](int i) { return HalfRef{x[i / 2], (i & 1) != 0}; }, half_lo(mn), half_lo(mx), j.mode,
                               a.sym_den_literal, words, s, z);
  // a row is one plane of LB-bit fields over all channels (3-bit: followed by the plane of high bits)
  constexpr int LB = BITS == 3 ? 2 : BITS;
  constexpr int WL = G * LB / 32;                        // words of the (low) plane of one group
  long long lin = (long long)bh * a.capacity + row0;     // first row of the unit (uniform), then the lane's from it
  uint32_t dr = r;
  if (a.pages.table) {
    lin = store_row(a.pages, a.n_kv_heads, a.capacity, bh, row0 + r);
    dr = 0u;
  }
  uint32_t* rowp = reinterpret_cast<uint32_t*>(j.codes + lin * (D * BITS / 8)) + dr * (D * BITS / 32);
#pragma unroll
  for (int i = 0; i < WL; i += 2) *reinterpret_cast<uint2*>(rowp + g * WL + i) = uint2{words[i], words[i + 1]};
  if constexpr (BITS == 3) {
#pragma unroll
    for (int i = 0; i < G / 32; ++i) rowp[D * 2 / 32 + g * (G / 32) + i] = words[WL + i];
  }
  (j.scales + lin * GPR)[dr * GPR + g] = s;
  if (j.zeros) (j.zeros + lin * GPR)[dr * GPR + g] = z;
}

// ---- per-channel form ----------------------------------------------------------------------
// One group of G tokens (tg) of sequence-head bh, all channels; or (RING) 128 / G groups from tg on, one channel
// slice.  Groups from tg_end on are not there: their lanes repeat the last one, store included.
template <int BITS, bool RING>
__device__ __forceinline__ void per_channel_unit(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t tg,
                                                 uint32_t tg_end, uint32_t slice) {
  constexpr int W = G * BITS / 32;
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t c = 2u * lane, dt = 0u;                       // channel pair; group, counted from tg
  if (RING) {
    c = slice * G + 2u * (lane % (G / 2));
    dt = lane / (G / 2);
    dt = tg + dt < tg_end ? dt : tg_end - 1u - tg;
  }
  const long long t0 = (long long)a.w_sink + (long long)(tg + dt) * G;
  const uint32_t* base = reinterpret_cast<const uint32_t*>(
      j.x_new + ((long long)bh * a.t_new + ((long long)a.w_sink + (long long)tg * G - a.n_old)) * D);      // (uniform)
  const uint32_t* src = base + (dt * (G * D / 2) + c / 2);
  uint32_t x[G];
  if constexpr (!RING) {
#pragma unroll
    for (int i = 0; i < G; ++i) x[i] = src[i * (D / 2)];
  } else {
    const uint32_t* ring = reinterpret_cast<const uint32_t*>(j.ring + (long long)bh * j.slots * D + c);
    uint32_t slot = (uint32_t)t0 % (uint32_t)j.slots;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const uint32_t* p = t0 + i >= a.n_old ? src + i * (D / 2) : ring + slot * (D / 2);
      x[i] = *p;
      slot = slot + 1u == (uint32_t)j.slots ? 0u : slot + 1u;
    }
  }
  if (j.normalise) {
    const float* inv = a.inv_norm + (bh % (uint32_t)a.n_kv_heads) * D + c;
    const float f0 = inv[0], f1 = inv[1];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const uint32_t y = scaled_pair(x[i], f0, f1);
      x[i] = !RING || t0 + i >= a.n_old ? y : x[i];      // (ring rows already are)
    }
  }
  uint32_t mn, mx;
  pair_range(x, mn, mx);
  uint32_t words[2][W];
  __half s[2], z[2];
  quantize_group_bulk<G, BITS>([&](int i) { return HalfRef{x[i], false}; }, half_lo(mn), half_lo(mx), j.mode,
                               a.sym_den_literal, words[0], s[0], z[0]);
  quantize_group_bulk<G, BITS>([&](int i) { return HalfRef{x[i], true}; }, half_hi(mn), half_hi(mx), j.mode,
                               a.sym_den_literal, words[1], s[1], z[1]);
  long long go = ((long long)bh * a.capacity / G + tg) * D;            // (capacity is a multiple of G)
  uint32_t dc = dt * D + c;
  if (a.pages.table) {
    go = (store_row(a.pages, a.n_kv_heads, a.capacity, bh, (long long)(tg + dt) * G) / G) * D;
    dc = c;
  }
  uint32_t* dst = reinterpret_cast<uint32_t*>(j.codes) + go * W + dc * W;   // 2 W words from an even channel: 8-byte aligned
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const uint32_t w0 = 2 * i < W ? words[0][2 * i] : words[1][2 * i - W];
    const uint32_t w1 = 2 * i + 1 < W ? words[0][2 * i + 1] : words[1][2 * i + 1 - W];
    *reinterpret_cast<uint2*>(dst + 2 * i) = uint2{w0, w1};
  }
  auto pair = [](__half lo, __half hi) { return (uint32_t)__half_as_ushort(lo) | ((uint32_t)__half_as_ushort(hi) << 16); };
  *reinterpret_cast<uint32_t*>(j.scales + go + dc) = pair(s[0], s[1]);
  if (j.zeros) *reinterpret_cast<uint32_t*>(j.zeros + go + dc) = pair(z[0], z[1]);
}

// Rows (store rows) of a job that come from the ring and from the new tokens.
struct Split { long long ring, fresh; };
__host__ __device__ inline Split split_rows(const QuantArgs& a, const QuantTensorJob& j) {
  const long long rows = j.row_end > j.row_begin ? j.row_end - j.row_begin : 0;
  long long old = a.n_old - a.w_sink - j.row_begin;      // of them are older than this call
  old = old < 0 ? 0 : old;
  if (j.form == kPerChannel) old = (old + G - 1) / G * G;
  old = old > rows ? rows : old;
  return {old, rows - old};
}

// New tokens to their windows, one channel slice of one sequence-head (see window_copy).
__device__ __forceinline__ void copy_slice(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t slice) {
  constexpr uint32_t PER_ROW = G / 8;                    // 16-byte pieces of a slice's row
  const CopySpan sp = copy_span(a, j);
  const uint32_t n_a = (uint32_t)sp.n_a, n = (uint32_t)(sp.n_a + (a.t_new - sp.i_b)) * PER_ROW;
  const uint32_t c = slice * G + 8u * (threadIdx.x % PER_ROW);
  for (uint32_t at = threadIdx.x; at < n; at += 1024u) {
    uint4 raw[4];
    __half* dst[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {                        // (the loads of four rows go out together)
      const uint32_t idx = at + 256u * p < n ? at + 256u * p : at;
      const uint32_t k = idx / PER_ROW;
      const long long i = k < n_a ? (long long)k : sp.i_b + (k - n_a), t = a.n_old + i;
      dst[p] = (t < a.w_sink ? j.sink + ((long long)bh * a.w_sink + t) * D
                             : j.ring + ((long long)bh * j.slots + (uint32_t)t % (uint32_t)j.slots) * D) + c;
      raw[p] = *reinterpret_cast<const uint4*>(j.x_new + ((long long)bh * a.t_new + i) * D + c);
    }
    if (j.normalise) {
      const float* inv = a.inv_norm + (bh % (uint32_t)a.n_kv_heads) * D + c;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        raw[p].x = scaled_pair(raw[p].x, inv[0], inv[1]);
        raw[p].y = scaled_pair(raw[p].y, inv[2], inv[3]);
        raw[p].z = scaled_pair(raw[p].z, inv[4], inv[5]);
        raw[p].w = scaled_pair(raw[p].w, inv[6], inv[7]);
      }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) *reinterpret_cast<uint4*>(dst[p]) = raw[p];
  }
}

constexpr uint32_t kSlices = D / G;                      // channel slices, and groups per row
constexpr uint32_t kUnitRows = 64u / kSlices;            // rows of a per-token unit

struct BulkPlan {
  uint32_t ring_groups;                                  // work-groups in front that own a ring slice each: 2 BH kSlices
  uint32_t per_bh_t, per_bh_c;                           // units per sequence-head of the per-token / per-channel tensor
};

template <int BITS>
__device__ __forceinline__ void ring_units(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t slice,
                                           uint32_t row0, uint32_t rows) {
  const uint32_t wave = threadIdx.x >> 6;
  if (j.form == kPerToken) {
    for (uint32_t r = 64u * wave; r < rows; r += 256u) per_token_unit<BITS, true>(a, j, bh, row0 + r, row0 + rows, slice);
  } else {
    constexpr uint32_t PER = 128u / G;                   // groups a wavefront takes
    const uint32_t tg0 = row0 / G, n = rows / G;
    for (uint32_t t = PER * wave; t < n; t += 4u * PER) per_channel_unit<BITS, true>(a, j, bh, tg0 + t, tg0 + n, slice);
  }
}

template <bool INNER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 32 ? 4 : 3))) quantize_bulk_kernel(QuantArgs a, BulkPlan p) {
  if (blockIdx.x < p.ring_groups) {
    // ---- a ring slice: what leaves it, then what enters
    const uint32_t slice = blockIdx.x % kSlices, tensor = (blockIdx.x / kSlices) & 1u, bh = blockIdx.x / (2u * kSlices);
    const QuantTensorJob j = pick_job(a, (int)tensor);
    const uint32_t rows = (uint32_t)split_rows(a, j).ring;
    if (rows > 0u) {
      if (j.bits == 2) ring_units<2>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
      else if (j.bits == 3) ring_units<3>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
      else ring_units<4>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
    }
    __syncthreads();                                     // every row of this slice has been read
    copy_slice(a, j, bh, slice);
    return;
  }
  const uint32_t BH = (uint32_t)(a.batch * a.n_kv_heads);
  uint32_t u = __builtin_amdgcn_readfirstlane((blockIdx.x - p.ring_groups) * 4u + (threadIdx.x >> 6));
  if (u < BH * p.per_bh_t) {
    const QuantTensorJob j = pick_job(a, INNER ? 0 : 1);
    const uint32_t bh = u / p.per_bh_t, row0 = (uint32_t)(j.row_begin + split_rows(a, j).ring) + (u - bh * p.per_bh_t) * kUnitRows;
    const uint32_t row_end = (uint32_t)j.row_end;
    if (j.bits == 2) per_token_unit<2, false>(a, j, bh, row0, row_end, 0u);
    else if (j.bits == 3) per_token_unit<3, false>(a, j, bh, row0, row_end, 0u);
    else per_token_unit<4, false>(a, j, bh, row0, row_end, 0u);
    return;
  }
  u -= BH * p.per_bh_t;
  if (u < BH * p.per_bh_c) {
    const QuantTensorJob j = pick_job(a, INNER ? 1 : 0);
    const uint32_t bh = u / p.per_bh_c, tg = (uint32_t)((j.row_begin + split_rows(a, j).ring) / G) + (u - bh * p.per_bh_c);
    if (j.bits == 2) per_channel_unit<2, false>(a, j, bh, tg, tg + 1u, 0u);
    else if (j.bits == 3) per_channel_unit<3, false>(a, j, bh, tg, tg + 1u, 0u);
    else per_channel_unit<4, false>(a, j, bh, tg, tg + 1u, 0u);
  }
}

}  // namespace

#if INNERQ_BULK_GROUP == 32
bool bulk_append_supported(const QuantArgs& a) {
  if (a.n_dev || a.t_new < 2) return false;
  long long most = 0;
  bool shared = false;                                   // a new token lands in a ring slot that this call reads
  for (int w = 0; w < 2; ++w) {
    const QuantTensorJob& j = a.job[w];
    if (j.form == kFp16) return false;
    const long long groups = (long long)a.batch * a.n_kv_heads * (j.row_end - j.row_begin) * (D / a.group);
    // (a launch's index arithmetic is 32-bit)
    if (groups + 64 >= (1LL << 32) || j.row_end >= (1LL << 31) || a.n_old + a.t_new >= (1LL << 31)) return false;
    most = groups > most ? groups : most;
    shared = shared || ring_slots_shared(a, j);
  }
  // The other form (launch_quantize_t) spreads a group over eight lanes, which is the shorter chain while the chip is
  // idle, but needs a second launch when ring slots are shared.  Per call, 8 kv heads: 128 tokens onto 500 cached
  // ones 7.5 us against 10.0; a first 400 tokens (12800 groups) 5.1 against 5.1, a first 1000 (32000 groups) 5.2
  // against 7.2.  With more ring work-groups than fit at once the second launch is the cheaper one: 32 sequences, 8
  // tokens each (8192 groups) 9.5 against 6.5.
  const bool few_rings = 2LL * a.batch * a.n_kv_heads * (D / a.group) <= 4LL * compute_units();
  return most >= 16384 || (most > 0 && shared && few_rings);
}

hipError_t launch_quantize_bulk_g64(const QuantArgs& a, hipStream_t stream);
hipError_t launch_quantize_bulk(const QuantArgs& a, hipStream_t stream) {
  if (a.group == 64) return launch_quantize_bulk_g64(a, stream);
#else
hipError_t launch_quantize_bulk_g64(const QuantArgs& a, hipStream_t stream) {
#endif
  if (a.group != G) return hipErrorInvalidValue;
  const bool inner = a.job[0].form == kPerToken;
  const long long BH = (long long)a.batch * a.n_kv_heads;
  const QuantTensorJob &jt = a.job[inner ? 0 : 1], &jc = a.job[inner ? 1 : 0];
  const long long per_bh_t = (split_rows(a, jt).fresh + kUnitRows - 1) / kUnitRows, per_bh_c = split_rows(a, jc).fresh / G;
  const long long ring_groups = 2 * BH * kSlices, blocks = (BH * (per_bh_t + per_bh_c) + 3) / 4;
  const BulkPlan p = {(uint32_t)ring_groups, (uint32_t)per_bh_t, (uint32_t)per_bh_c};
  const unsigned grid = (unsigned)(ring_groups + blocks);
  if (inner) quantize_bulk_kernel<true><<<grid, 256, 0, stream>>>(a, p);
  else quantize_bulk_kernel<false><<<grid, 256, 0, stream>>>(a, p);
  return hipGetLastError();
}

}  // namespace innerq

// Chunks onto a filled cache in one launch: quantise, pack and copy into the windows, where a new token lands in a
// ring slot that the same call still has to read.
//
// A work-group owns a slice of G channels of one ring (of one sequence-head and tensor): it quantises the tokens that
// leave the slice and, behind a barrier, writes the tokens that enter it, so no second launch has to wait for the first.
// New tokens that do not stay in a window are units of one wavefront each:
//   * per-token form: 64 consecutive groups of one sequence-head, one a lane (its G channels are 2 G contiguous bytes,
//     and the 64 lanes' loads and packed stores are contiguous too);
//   * per-channel form: half of the channels of one group of G tokens, a lane a channel (a token's row is coalesced 128-byte loads);
//     or, in a kernel of its own (PAIRS), all of them, a lane a pair.
//
// What bounds it is the chain of an owner: the rounds of loads of the rows that leave, one lane's whole group, the
// rounds of copies.  It pays while the owners fit the chip and their rings are short (append_form): 512 tokens onto 500 of 8 heads, G = 32, 6.2 us against 8.6 in two launches; 32 heads 7.8
// against 10.3; but with a window of 1024 tokens 19 against 10, and 157 against 13 with 8192 (1 head, G = 64): a ring's
// rows are one work-group's serial rounds.
#include "innerq_dev.h"
#include "quant_group.h"

#ifndef INNERQ_OWNERS_GROUP
#define INNERQ_OWNERS_GROUP 32
#endif

namespace innerq {
namespace {

constexpr int G = INNERQ_OWNERS_GROUP;
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
  long long lin = (long long)bh * a.capacity + row0;     // first row of the unit (uniform), then the lane's from it
  uint32_t dr = r;
  if (a.pages.table) {
    lin = store_row(a.pages, a.n_kv_heads, a.capacity, bh, row0 + r);
    dr = 0u;
  }
  per_token_group<G, BITS, false>(a, j, src, !RING || fresh, bh, g, lin, dr);
}

// ---- per-channel form ----------------------------------------------------------------------
// One group of G tokens (tg) of sequence-head bh, half of the channels (part), a lane each; or (RING) 64 / G groups from tg on, one
// channel slice (part).  PAIR: two channels a lane, one after the other: all channels, or twice the groups.  Groups from tg_end
// on are not there: their lanes repeat the last one, store included.
// A channel a lane is the shorter chain: 512 tokens onto 500 of 32 heads at 4 bits 7.8 us a chunk, with pairs alone 9.5; 250 of 32 heads,
// 3 bits, 7.3, 9.6; chunks of 8192 tokens of 32 heads 37, 39.  A pair is half the loads, which is what counts where a lane has 64 of
// them and one variant to compute (G = 64, 2 bits: 110 heads, 8583 tokens 162 us a channel a lane, 84 a pair), and one
// round of a ring's wavefronts where a channel a lane takes two (4 heads, 330 tokens, a window of 416, G = 32 8.3, 7.0; 1 head, 395, G = 64
// 12.7, 10.4).
template <int BITS, bool RING, bool PAIR>
__device__ __forceinline__ void per_channel_unit(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t tg,
                                                 uint32_t tg_end, uint32_t part) {
  constexpr int W = G * BITS / 32, C = PAIR ? 2 : 1;
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t c = PAIR ? 2u * lane : 64u * part + lane, dt = 0u;   // (first) channel; group, counted from tg
  if (RING) {
    c = part * G + C * (lane % (G / C));
    dt = lane / (G / C);
    dt = tg + dt < tg_end ? dt : tg_end - 1u - tg;
  }
  const long long t0 = (long long)a.w_sink + (long long)(tg + dt) * G;
  const __half* src = j.x_new + ((long long)bh * a.t_new + ((long long)a.w_sink + (long long)tg * G - a.n_old)) * D      // (uniform)
                      + (dt * (G * D) + c);
  auto load = [](const __half* p) { return PAIR ? *reinterpret_cast<const uint32_t*>(p) : (uint32_t)__half_as_ushort(*p); };
  uint32_t x[G];                                         // one value, in the low half, or two
  if constexpr (!RING) {
#pragma unroll
    for (int i = 0; i < G; ++i) x[i] = load(src + i * D);
  } else {
    const __half* ring = j.ring + (long long)bh * j.slots * D + c;
    uint32_t slot = (uint32_t)t0 % (uint32_t)j.slots;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      x[i] = load(t0 + i >= a.n_old ? src + i * D : ring + slot * D);
      slot = slot + 1u == (uint32_t)j.slots ? 0u : slot + 1u;
    }
  }
  if (j.normalise) {
    const float* f = a.inv_norm + (bh % (uint32_t)a.n_kv_heads) * D + c;
    const float f0 = f[0], f1 = PAIR ? f[1] : 0.f;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const uint32_t y = scaled_pair(x[i], f0, f1);
      x[i] = !RING || t0 + i >= a.n_old ? y : x[i];      // (ring rows already are)
    }
  }
  uint32_t mn, mx, words[C][W];
  pair_range(x, mn, mx);
  __half s[C], z[C];
  quantize_group_bulk<G, BITS, false>([&](int i) { return HalfRef{x[i], false}; }, NoDistances{}, half_lo(mn), half_lo(mx), j.mode,
                               a.sym_den_literal, words[0], s[0], z[0]);
  if constexpr (PAIR)
    quantize_group_bulk<G, BITS, false>([&](int i) { return HalfRef{x[i], true}; }, NoDistances{}, half_hi(mn), half_hi(mx), j.mode,
                                 a.sym_den_literal, words[1], s[1], z[1]);
  long long go = ((long long)bh * a.capacity / G + tg) * D;            // (capacity is a multiple of G)
  uint32_t dc = dt * D + c;
  if (a.pages.table) {
    go = (store_row(a.pages, a.n_kv_heads, a.capacity, bh, (long long)(tg + dt) * G) / G) * D;
    dc = c;
  }
  uint32_t* dst = reinterpret_cast<uint32_t*>(j.codes) + go * W + dc * W;
  if constexpr (PAIR) {                                                  // 2 W words from an even channel: 8-byte aligned
#pragma unroll
    for (int i = 0; i < C * W; i += 2) *reinterpret_cast<uint2*>(dst + i) = uint2{words[i / W][i % W], words[(i + 1) / W][(i + 1) % W]};
    auto both = [](const __half (&x)[C]) { return (uint32_t)__half_as_ushort(x[0]) | (uint32_t)__half_as_ushort(x[C - 1]) << 16; };
    *reinterpret_cast<uint32_t*>(j.scales + go + dc) = both(s);
    if (j.zeros) *reinterpret_cast<uint32_t*>(j.zeros + go + dc) = both(z);
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) dst[i] = words[0][i];
    (j.scales + go)[dc] = s[0];
    if (j.zeros) (j.zeros + go)[dc] = z[0];
  }
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

struct OwnersPlan {
  uint32_t ring_groups;                                  // work-groups in front that own a ring slice each: 2 BH kSlices
  uint32_t per_bh_t, per_bh_c;                           // units per sequence-head of the per-token / per-channel tensor
};

// PAIRS: two channels a lane in every unit of the per-channel tensor; else one, in a ring of G = 64 of at most four groups
// (the launch sees to it).
template <int BITS, bool PAIRS>
__device__ __forceinline__ void ring_units(const QuantArgs& a, const QuantTensorJob& j, uint32_t bh, uint32_t slice,
                                           uint32_t row0, uint32_t rows) {
  const uint32_t wave = threadIdx.x >> 6;
  if (j.form == kPerToken) {
    for (uint32_t r = 64u * wave; r < rows; r += 256u) per_token_unit<BITS, true>(a, j, bh, row0 + r, row0 + rows, slice);
  } else {
    constexpr uint32_t PER = 64u / G;                    // groups a wavefront takes
    const uint32_t tg0 = row0 / G, n = rows / G;
    if (!PAIRS && (G == 64 || n <= 4u * PER)) {
      // (no loop: 8 heads, 512 tokens onto 500, G = 32 6.2 us a chunk, with one 6.7)
      if (PER * wave < n) per_channel_unit<BITS, true, false>(a, j, bh, tg0 + PER * wave, tg0 + n, slice);
    } else {
      for (uint32_t t = 2u * PER * wave; t < n; t += 8u * PER) per_channel_unit<BITS, true, true>(a, j, bh, tg0 + t, tg0 + n, slice);
    }
  }
}

template <bool INNER, bool PAIRS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 32 ? 4 : 3))) quantize_owners_kernel(QuantArgs a, OwnersPlan p) {
  if (blockIdx.x < p.ring_groups) {
    // ---- a ring slice: what leaves it, then what enters
    const uint32_t slice = blockIdx.x % kSlices, tensor = (blockIdx.x / kSlices) & 1u, bh = blockIdx.x / (2u * kSlices);
    const QuantTensorJob j = pick_job(a, (int)tensor);
    const uint32_t rows = (uint32_t)split_rows(a, j).ring;
    if (rows > 0u) {
      if (j.bits == 2) ring_units<2, PAIRS>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
      else if (j.bits == 3) ring_units<3, PAIRS>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
      else ring_units<4, PAIRS>(a, j, bh, slice, (uint32_t)j.row_begin, rows);
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
    const uint32_t bh = u / p.per_bh_c, at = u - bh * p.per_bh_c;
    const uint32_t first = (uint32_t)((j.row_begin + split_rows(a, j).ring) / G);
    const uint32_t tg = first + (PAIRS ? at : at >> 1), part = PAIRS ? 0u : at & 1u;
    if (j.bits == 2) per_channel_unit<2, false, PAIRS>(a, j, bh, tg, tg + 1u, part);
    else if (j.bits == 3) per_channel_unit<3, false, PAIRS>(a, j, bh, tg, tg + 1u, part);
    else per_channel_unit<4, false, PAIRS>(a, j, bh, tg, tg + 1u, part);
  }
}

}  // namespace

#if INNERQ_OWNERS_GROUP == 32
// One chunk measured in its form and without owners, 23000 drawn shapes that meet the first line of the rule below (sequence-heads,
// tokens and windows over their ranges, all widths and modes, both group sizes).
AppendForm append_form(const QuantArgs& a) {
  if (a.n_dev) return AppendForm::kLanes8;
  long long most = 0, slice_rows = 0, ring_groups = 0;
  int channel_bits = 2;
  bool shared = false, values = false, ring_values = false, hybrid = false, both = false;
  bool narrow = a.n_old + a.t_new < (1LL << 31);         // (the owners' row arithmetic is 32-bit)
  for (int w = 0; w < 2; ++w) {
    const QuantTensorJob& j = a.job[w];
    if (j.form == kFp16) return AppendForm::kLanes8;
    const long long rows = j.row_end - j.row_begin, groups = (long long)a.batch * a.n_kv_heads * rows * (D / a.group);
    narrow = narrow && groups + 64 < (1LL << 32);
    most = groups > most ? groups : most;
    shared = shared || ring_slots_shared(a, j);
    hybrid = hybrid || j.mode == INNERQ_HYBRID;
    if (j.form == kPerChannel) {
      values = rows > 0;
      channel_bits = j.bits;
      both = j.mode == INNERQ_HYBRID;
      ring_values = rows > 0 && a.w_sink + j.row_begin < a.n_old;
    }
    // rows that an owner reads from its ring, tokens that it writes
    long long old = a.n_old - a.w_sink - j.row_begin;
    old = old < 0 ? 0 : old > rows ? rows : old;
    if (j.form == kPerChannel) ring_groups = (old + a.group - 1) / a.group;
    const CopySpan sp = copy_span(a, j);
    const long long in = sp.n_a + (a.t_new - sp.i_b);
    slice_rows = old > slice_rows ? old : slice_rows;
    slice_rows = in > slice_rows ? in : slice_rows;
  }
  // Owners of ring slices: where per-channel groups leave a ring (a chunk that only moves keys on is a short chain in
  // either form: 16 heads, 8 tokens 5.0 us in two launches of eight lanes a group, 5.3 here), at most two owners a
  // compute unit (64 x 8 heads, 8 tokens 17 us here, 7.7 there) and rings of up to 448 rows (above).  The time without them, by groups (ratio
  // of geometric means): G = 32, both variants to 8192 1.03, to 32768 1.30, to 131072 1.23, to 512k 1.16, to 2 M 1.06; one
  // variant 1.20, 1.35, 1.31, 1.18, 1.08.  Beyond, to 3 M, 4 M, 8 M and more, two launches and a channel a lane over pairs: both, 2 bits 1.05 1.02, 1.04 1.04,
  // 1.00 1.05, 0.99 1.05; 3 bits 1.06 1.01, 1.05 1.02, 1.04 1.02, 1.05 1.03; 4 bits 1.03 1.02, 0.99 1.05, 0.98 1.05, 1.00 1.08; one, 2 bits 1.05 0.97,
  // 1.01 0.99, 1.01 0.97, 1.01 0.97; 3 bits 1.02 1.02, 0.97 1.06, 1.01 0.99, 1.02 0.98; 4 bits 1.04 0.99, 1.01 1.01, 1.03 0.98, 1.02 0.98.
  // At G = 64 a lane's chain is twice as long.  Time relative to the best of three forms (two launches / owners, a channel a lane / owners,
  // pairs), geometric means of 6000 drawn chunks, by groups of the larger tensor up to
  //                                        2048            8192            65536           131072          262144          512k            more
  //   one variant, 2 bits             1.00 1.06 1.35  1.23 1.02 1.30  1.43 1.00 1.21  1.24 1.08 1.00  1.16 1.25 1.00  1.07 1.31 1.00  1.00 1.45 1.01
  //   one variant, 3 bits             1.00 1.13 1.49  1.22 1.05 1.37  1.41 1.00 1.24  1.19 1.00 1.06  1.04 1.05 1.00  1.00 1.12 1.03  1.00 1.32 1.09
  //   one variant, 4 bits             1.00 1.10 1.37  1.21 1.04 1.29  1.43 1.00 1.21  1.27 1.00 1.07  1.01 1.00 1.04  1.00 1.12 1.10  1.00 1.28 1.21
  //   both variants, 2 bits           1.00 1.28 1.79  1.00 1.23 1.72  1.34 1.00 1.30  1.02 1.00 1.02  1.00 1.12 1.01  1.00 1.19 1.02  1.00 1.44 1.04
  //   both variants, 3 and 4 bits     1.00 1.35 1.90  1.00 1.29 1.81  1.32 1.00 1.32  1.06 1.00 1.16  1.00 1.00 1.10  1.00 1.06 1.08  1.00 1.19 1.08
  // and, of pairs alone, where a ring's groups are more than one round of its wavefronts (two launches over pairs): one variant 1.08 to 1.20
  // from 8192 groups to 512k, beyond 1.02 at 2 bits and 0.93 at 3 and 4; both, from 24 heads on, 1.06 to 1.12 up to 196608, fewer heads 0.99.
  const long long heads = (long long)a.batch * a.n_kv_heads, owners = 2 * heads * (D / a.group);
  const bool few_short = narrow && owners <= 2LL * compute_units() && slice_rows <= 448;
  if (few_short && shared && ring_values && a.group == 32) {
    return most >= 2097152 && (hybrid || channel_bits == 3) ? AppendForm::kRingOwnersPairs : AppendForm::kRingOwners;
  } else if (few_short && shared && ring_values) {
    const bool one_round = ring_groups <= 4;
    const long long from = one_round && !both ? 3072 : 8192;
    const long long single_to = !one_round ? 0 : both ? (channel_bits == 2 ? 98304 : 163840) : 65536 * (channel_bits - 1);
    const long long pairs_to = both ? (!one_round && heads >= 24 ? 196608 : 0) : channel_bits == 2 ? 1048576 : !one_round ? 524288 : channel_bits == 3 ? 262144 : 0;
    if (most >= from && most < single_to) return AppendForm::kRingOwners;
    if (most >= from && most < pairs_to) return AppendForm::kRingOwnersPairs;
  }
  // A group a lane, or spread over eight: the chain of a lane's group is the longer one, but eight lanes are eight times the
  // wavefronts (a first prompt of hybrid groups, G = 32, 4 bits: 4 heads, 600 tokens (7488 groups) 4.2 us against 4.7, 16 heads, 300
  // (10752) 5.1 against 4.8; G = 64: 8 heads, 600 (7488) 4.8 against 6.4, 1000 (13888) 6.3 against 6.0; 3-bit symmetric ones 4.2 against 4.0 at
  // 5376), or, with nothing but keys, as long as there are wavefronts to spare: a single token of 8192 heads (32768 groups) 7.0
  // against 5.9, of 2048 heads the same; beside the second launch of a chunk longer (2048 heads, 2 tokens (16384 groups) 7.5 against
  // 9; 8 tokens 10.2 against 10.5).
  return most < (values ? (hybrid ? 8192 : 4096) : shared ? 65536 : 16384) ? AppendForm::kLanes8 : AppendForm::kLane;
}

hipError_t launch_quantize_owners_g64(const QuantArgs& a, bool pairs, hipStream_t stream);
hipError_t launch_quantize_owners(const QuantArgs& a, bool pairs, hipStream_t stream) {
  if (a.group == 64) return launch_quantize_owners_g64(a, pairs, stream);
#else
hipError_t launch_quantize_owners_g64(const QuantArgs& a, bool pairs, hipStream_t stream) {
#endif
  if (a.group != G) return hipErrorInvalidValue;
  const bool inner = a.job[0].form == kPerToken;
  const long long BH = (long long)a.batch * a.n_kv_heads;
  const QuantTensorJob &jt = a.job[inner ? 0 : 1], &jc = a.job[inner ? 1 : 0];
  if (G == 64 && !pairs && split_rows(a, jc).ring > 4 * G) return hipErrorInvalidValue;      // (see ring_units)
  const long long per_bh_t = (split_rows(a, jt).fresh + kUnitRows - 1) / kUnitRows, per_bh_c = split_rows(a, jc).fresh / G * (pairs ? 1 : 2);
  const long long ring_groups = 2 * BH * kSlices, blocks = (BH * (per_bh_t + per_bh_c) + 3) / 4;
  const OwnersPlan p = {(uint32_t)ring_groups, (uint32_t)per_bh_t, (uint32_t)per_bh_c};
  const unsigned grid = (unsigned)(ring_groups + blocks);
  if (pairs) {
    if (inner) quantize_owners_kernel<true, true><<<grid, 256, 0, stream>>>(a, p);
    else quantize_owners_kernel<false, true><<<grid, 256, 0, stream>>>(a, p);
    return hipGetLastError();
  }
  if (inner) quantize_owners_kernel<true, false><<<grid, 256, 0, stream>>>(a, p);
  else quantize_owners_kernel<false, false><<<grid, 256, 0, stream>>>(a, p);
  return hipGetLastError();
}

}  // namespace innerq

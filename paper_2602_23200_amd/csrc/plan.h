// The launch plan of an attention call: how the tokens go to wavefronts, work-groups and window chunks, and whether the
// launch joins its own partial results.  Host arithmetic on sizes alone (no HIP), so that every plan can be checked without a
// device.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "../../include/innerq.h"

namespace innerq {

constexpr int kHeadDim = 128;          // the only head_dim built
constexpr int kWindowChunk = 64;       // most window tokens per wavefront / work-group chunk
constexpr int kWindowChunkMin = 16;    // fewest (short contexts, slots to spare)
constexpr int kHeadTile = 4;           // query heads served by one work-group pass
constexpr int kShortTokens = 256;      // most tokens of a cache that one work-group attends to by itself (attention_generic.hip)

constexpr int kJoinWaves = 8;            // most wavefronts of a work-group that joins its own
constexpr int kJoinGroups = 8;           // most work-groups of a sequence-head that join (one round of loads brings eight partials)
// bytes of one partial of one head: 128 channels, and level and sum for each half of them
constexpr int kJoinBytes = (kHeadDim + 4) * 8;

inline long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

// Most window chunks a launch may use (chunks of kWindowChunkMin tokens); bounds the workspace.
inline int window_chunk_cap(const innerq_config_t& c) {
  return (int)ceil_div((long long)c.w_sink + c.w_recent + 2LL * c.group, kWindowChunkMin) + 1;
}
// Most token splits a launch may use for the quantised range; bounds the workspace.  Never below
// the window chunk count plus one: the fused inner kernel needs one wavefront beyond those that
// carry a window chunk.
inline int split_cap(const innerq_config_t& c) {
  long long s = ceil_div(4096, (long long)c.batch * c.n_kv_heads);
  if (s < 4) s = 4;
  if (s > 512) s = 512;
  if (s < window_chunk_cap(c) + 1) s = window_chunk_cap(c) + 1;
  return (int)s;
}

// Bytes at the start of the workspace for one int per sequence: the fused kernel of a ragged step leaves
// the sequences' token counts there for the append that follows it -- and, for batches that share the launch's
// wavefronts by length, behind them how many partial results each sequence has (these fit the first 256 bytes).
constexpr int kSharedBatchMost = 32;
inline size_t seq_bytes(const innerq_config_t& c) { return (((size_t)c.batch * sizeof(int) + 255) / 256) * 256; }
static_assert(2 * kSharedBatchMost * sizeof(int) <= 256, "both counts of a sequence in the first 256 bytes");

enum FusedKind : int { kFp32Kernel = 0, kInnerKernel = 1, kFp16Kernel = 2, kOuterKernel = 3 };

struct PlanInput {
  int fused_kind;               // FusedKind: the kernel that serves the quantised range
  int compute_units, waves_per_cu;
  bool may_join;                // the kernel can join its own partials
  bool appends;                 // the launch would take a decode step's append along
  bool spills;                  // the append of a step over these tokens moves a value group out of its ring
  bool ragged;                  // token counts on the device: n_both, win_tokens hold for the longest sequence allowed
  long long n_both;             // tokens of the quantised range
  long long win_tokens;         // tokens outside it
  int tile_tokens = 64;         // of a tile of the kernel
};

// Grid of the outer-grouped kernel: sequence-heads, then the parts of one (window chunks and token ranges), which are more than a
// grid's second dimension can be (65536) where the window is longer than a million tokens: the rest goes to the third.  A part is
// z * kGridParts + y; of the last layer some are not there.
constexpr int kGridParts = 32768;
struct HeadsByParts { unsigned x, y, z; };
inline HeadsByParts heads_by_parts(long long heads, long long parts) {
  return {(unsigned)heads, (unsigned)(parts < kGridParts ? parts : kGridParts), (unsigned)ceil_div(parts, kGridParts)};
}

struct LaunchPlan {
  int n_splits;                 // wavefronts (fp32 kernel: work-groups) of a sequence-head that share the quantised range; 0: there is none
  int n_win;                    // window chunks
  int waves;                    // wavefronts per work-group
  int n_partials;               // partial results of a head
  int shared_groups;            // ragged: work-groups of a kv head shared by the sequences' lengths; 0: the same number each
  bool joins;                   // the launch joins its partials itself
  size_t workspace_bytes;       // of the call
};

inline LaunchPlan plan_attention(const innerq_config_t& c, const PlanInput& in) {
  const int kb = c.bits, vb = c.v_bits ? c.v_bits : c.bits, fused_kind = in.fused_kind;
  const long long n_both = in.n_both, win_tokens = in.win_tokens;
  const bool ragged = in.ragged, may_join = in.may_join;
  int n_partials = 0, shared_groups = 0;
  const int r = c.n_q_heads / c.n_kv_heads;
  int n_splits = 0, win_chunk_len = kWindowChunk, waves = 1;
  const bool fused = fused_kind != 0;
  const long long BH = (long long)c.batch * c.n_kv_heads;
  const bool can_join = fused_kind == kInnerKernel && n_both > 0 && !ragged && may_join;
  // A value group that leaves its ring (one step of G) takes a launch that the merge can share: there it is kept until the join
  // saves more than that (us of such a step, joined and with the merge: 2 heads x 6k tokens at 4 bits 17.7, 11.6, 8 x 8 x 4k 15.4,
  // 12.7, 16 x 8 x 8k 25.4, 23.9; 32 x 8 x 1k 19.5, 22.8).
  const bool with_the_group = in.spills && BH < in.compute_units;
  bool joins = can_join && !(with_the_group && in.appends);
  // Partial results a head may have where the launch joins them itself (they are larger there: kJoinBytes each).
  const long long most_groups = (long long)(split_cap(c) + window_chunk_cap(c)) * (kHeadDim + 2) * (long long)sizeof(float) / kJoinBytes;
  const bool heavy = kb == 3 || vb == 3;
  if (n_both > 0 && fused) {
    // one wavefront per split; every wavefront of the launch resident at once, no tail round
    // (the window wavefronts of the same launch take their share of the slots)
    const long long slots = (long long)in.compute_units * in.waves_per_cu;
    const long long n_tiles = ceil_div(n_both, in.tile_tokens);
    long long per_head = slots / ((long long)c.batch * c.n_kv_heads);
    // Short contexts: with fewer than about four tiles per wavefront, a launch of half as many
    // wavefronts (one per SIMD instead of two) is the faster one -- every wavefront pays its query
    // set-up once, and the launch itself costs time per wavefront (measured on the 32-head 4k-token
    // configuration, 4 bits: 17.8 -> 14.3 us per step; the two meet at four tiles per wavefront.  Eight query heads and 3-bit keys
    // go by the same line; they have not been measured apart).
    const bool few_tiles = n_tiles < 4 * per_head;
    if (fused_kind == 1 && few_tiles && per_head >= 8) per_head /= 2;
    // Window chunk length and the number of plain wavefronts.
    bool one_group = false;
    long long best_len = kWindowChunk, best_cost = -1, best_plain = 1;
    auto plain_for = [&](long long len) {
      const long long nw = ceil_div(win_tokens, len);
      long long plain = per_head - nw;
      if (plain > n_tiles) plain = n_tiles;
      // the workspace holds split_cap + window_chunk_cap partials; the inner kernel's wavefronts
      // that carry a window chunk count as splits too
      const long long most = fused_kind == 1 ? split_cap(c) - nw : split_cap(c);
      if (plain > most) plain = most;
      return plain < 1 ? 1 : plain;
    };
    if (fused_kind == 1) {
      // Inner kernel, as measured (a window chunk costs its wavefront about as much whatever its
      // length, so short chunks pay only where wavefront slots go begging): 16 tokens while the
      // whole launch fills at most a quarter of the SIMDs (4-head 512-token configuration: 10.4 us
      // per step against 10.8 at 64); 32 tokens for short contexts on a busy chip (8 x 8 heads at 2k
      // tokens: 12.5 us against 13.0 at 64 and 14.1 at 16); 64 tokens from about 3k tokens on
      // (32 heads at 4k tokens: 13.4 us against 14.1 at 32 and 15.0 at 16) and wherever the slots
      // are all needed for tiles.
      const long long simds = (long long)in.compute_units * 4;
      const long long waves16 = (long long)c.batch * c.n_kv_heads * (plain_for(kWindowChunkMin) + ceil_div(win_tokens, kWindowChunkMin));
      best_len = waves16 * 4 <= simds ? kWindowChunkMin : (n_tiles < 48 ? 32 : kWindowChunk);
      best_plain = plain_for(best_len);
      // A short context: one work-group per sequence-head, its wavefronts a window chunk or a tile or two each.  On an idle chip not with
      // more than two 3-bit tiles for a wavefront (8 heads x 0.5k tokens, G = 64 9.6 us with the merge, 11.0), nor an attention call
      // by itself for eight query heads (8 x 0.5k, 4 bits 11.8, 13.1): these keep the merge.  Up to four query heads it does not
      // depend on the append: a step and the separate calls that it replaces give the same bits there.
      const long long chunks32 = ceil_div(win_tokens, 32);
      if (joins && n_tiles + chunks32 <= 12 && chunks32 <= 7 && BH <= in.compute_units) {
        one_group = 2 * BH >= in.compute_units || !(heavy && n_tiles > 2 * (8 - chunks32));
        if (with_the_group || (r > 4 && 4 * BH < in.compute_units && !in.appends)) one_group = false;
        joins = one_group;
        if (one_group) {
          best_len = 32;
          best_plain = plain_for(32);
        }
      }
    } else {
      // Comparison kernels: 64 tokens when the wavefront slots are all needed for tiles (long
      // contexts: a chunk then hides behind the tile work), shorter when slots are to spare and the
      // window chunk would be the longest wavefront of the launch.  Costs in units of one tile of
      // one wavefront: a chunk of L tokens about 4 + 14 L / 64 (outer-grouped kernel, tiles of 2.9 us: 5 / 8 + 3 L / 128; 8 heads x
      // 8k tokens 11.0 us a call with chunks of 16, 12.3 of 32, 14.2 of 64; 16 x 8 heads x 6k, eight query heads, 188.5, 73.5, 53.1).
      for (long long len = kWindowChunk; len >= kWindowChunkMin; len /= 2) {
        const long long nw = ceil_div(win_tokens, len);
        const long long plain = plain_for(len);
        const long long tile_cost = ceil_div(n_tiles, plain) * 8, win_cost = !nw ? 0 : fused_kind == kOuterKernel ? 5 + 12 * len / 64 : 32 + 14 * len / 8;   // x 8
        const long long cost = tile_cost > win_cost ? tile_cost : win_cost;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best_len = len; best_plain = plain; }
      }
    }
    win_chunk_len = (int)best_len;
    const long long n_win_chunks = ceil_div(win_tokens, best_len);
    // the inner kernel's first wavefronts each carry a window chunk besides their tiles; the
    // comparison kernels run the window chunks as extra wavefronts of the same launch
    n_splits = (int)(fused_kind == 1 ? best_plain + n_win_chunks : best_plain);
    const long long cus = in.compute_units;
    if (joins) {
      // Wavefronts per work-group and work-groups per sequence-head, all resident at once.  The join costs the same for
      // two work-groups and for eight, and more beyond (another round of loads, and more that arrive at once).
      long long groups = 1;
      if (one_group) {
        waves = n_splits < 8 ? n_splits : 8;
      } else if (few_tiles) {
        // A chip that is not full, up to 160 tiles: eight work-groups at most, wavefronts with one to three tiles each (us per
        // step, with the merge -> now; kv heads x tokens: 1 x 4k 11.3 -> 9.6, 8 x 4k 12.6 -> 10.2, 8 x 8k 13.6 -> 10.9,
        // 16 x 8k 13.1 -> 11.1, 32 x 8k 13.6 -> 12.5; captured in a graph, without the host's time for a second launch, 1 x 4k
        // 10.0 -> 10.2, 8 x 8k 12.5 -> 11.5).  More tiles want more wavefronts a head than that (in a graph: 4 x 11k 12.1 -> 13.2,
        // 8 x 16k 13.6 -> 13.7).
        const long long full = slots / BH, half = 4 * cus / BH;
        const long long most = full < 64 ? full : 64;
        long long want = n_tiles * 2 / 3 + n_win_chunks;
        if (want > most) want = most;
        if (want <= n_win_chunks) want = n_win_chunks + 1;
        waves = 8;
        // (a wavefront a SIMD where that is two tiles each at most: 32 x 4k tokens at 4 bits 11.4, with more 12.2; 8k 13.8, 12.5)
        if (half <= 32 && n_win_chunks < half && n_tiles <= 2 * half) want = want < half ? want : half;
        if (want <= 32 && (BH * want <= 4 * cus || want / 4 * 4 > want / 8 * 8)) waves = 4;
        if (waves > want) waves = (int)want;
        groups = ceil_div(want, waves);
        while (groups > 1 && groups * waves > most && (groups - 1) * waves > n_win_chunks) --groups;
        // Work-groups of four for a wavefront a SIMD: a compute unit each, not two for some and one for others (56 heads x 2k, 280
        // work-groups: 1.12 of the time with the merge; 40 x 4k 1.16).
        if (waves == 4 && BH * groups > cus && BH * want <= 4 * cus && 4 * (cus / BH) > n_win_chunks) groups = cus / BH;
        // Not where a second round would begin, nor for wider codes two wavefronts a SIMD (96 heads x 1.3k at 4 bits 13.6 with
        // the merge, 16.1).
        const long long launched = BH * groups, tiles = BH * n_tiles;
        const bool narrow = kb + vb <= 4;
        if (launched > cus * (8 / waves) || (!narrow && launched * waves > 4 * cus)) joins = false;
        if (groups > 1) {
          // Eight heads' outputs are twice the join (72 heads x 2k tokens 17.3, 19.8; 96 x 0.9k 16.8, 19.0); 3-bit tiles want a
          // SIMD to themselves (10 heads x 0.9k 12.2, 14.8; 64 heads x 8k 23.1, 25.1).
          if (heavy || r > 4) joins = false;
          const long long plain = groups * waves - n_win_chunks;
          if (waves == 4) {
            // (two work-groups of four for a compute unit: 72 heads x 6k 1.09 of the time with the merge, for one or two query heads
            // 0.87 to 1.01; from 128 heads on 0.90 to 0.95)
            if (launched > cus && (2 * BH < cus ? r > 2 : 8 * launched < 14 * cus)) joins = false;
            // ... nor on a busy chip where the window chunks are most of it (128 heads x 0.9k 1.08, x 0.6k 0.87, G = 64 0.93) or leave the
            // others more than three tiles each (72 and 80 heads x 1.6k 1.07)
            if (4 * BH >= cus && ((c.group == 32 && n_tiles >= 10 && plain < n_win_chunks) || (2 * BH < cus && n_tiles > 3 * plain))) joins = false;
          }
          // Up to 50 heads the merge is the faster one where a SIMD has more than four tiles, two of wider codes (32 x 5k at 4 bits 1.07,
          // 32 x 9k 1.02), and everywhere beyond 160 (96) tiles a head.
          if (n_tiles > (narrow ? 160 : 96) || (5 * BH < cus && tiles > (narrow ? 16 : 8) * cus)) joins = false;
        }
      } else {
        long long best = 0;
        for (int w = 8; w >= 4; w /= 2) {                // (of fewer, every one of the launch would take part in the join)
          const long long fit = cus * (8 / w) / BH, all = ceil_div(n_splits, w), g = fit < all ? fit : all;
          if (g * w <= n_win_chunks) continue;
          // (several work-groups of four: 72 heads x 6k to 9k 1.08 of the time with the merge, 96 x 6k 1.06, eight query heads 1.13;
          // 160 heads 0.95 to 1.00)
          if (w == 4 && g > 1 && (2 * BH < cus || r > 4)) continue;
          const long long got = g * w < n_splits ? g * w : n_splits;
          if (got * 10 > best * 11) { best = got; waves = w; groups = g; }
        }
        if (best == 0) {
          // more wavefronts than fit at once: in rounds, where they are many (1024 heads x 4k tokens 85.3 -> 75.2; 320 heads x 3k
          // tokens 35.8 and 52.2) and the window chunks not most of it (1024 x 1k 39.8 and 50.1, x 3k 1.03 to 1.08 of the time)
          waves = n_splits < 8 ? n_splits : 8;
          groups = ceil_div(n_splits, waves);
          if (n_tiles < 48 || BH < 4 * cus) joins = false;
          best = n_splits;
        }
        // Work-groups of several wavefronts may leave slots empty: not where that is two fifths of a tile more for each of them (208
        // heads, eight wavefronts a head instead of nine: 16k tokens, 3.4 tiles more, 51.9 us -> 59.3; 112 heads, 16 instead of
        // 18: 6.5k tokens, 0.7 more, 18.5 -> 19.5).
        if (10 * n_tiles * (n_splits - best) > 4 * best * n_splits) joins = false;
      }
      if (groups > kJoinGroups || groups > most_groups) joins = false;
      // An attention call by itself gains less (there is no append to save) and keeps the merge on a chip that is not full
      // (4 heads x 9k tokens 11.7 us, joined 12.5) and with work-groups of four (160 heads x 3.6k tokens 18.8, 20.2).
      if (groups > 1 && (few_tiles || waves < 8) && !in.appends) joins = false;
      if (joins) {
        n_splits = (int)(groups * waves);
        n_partials = (int)groups;
      }
    }
    if (can_join && !joins) {
      // Four wavefronts that share the query tables are worth it for eight heads of narrow codes on a chip of one wavefront a
      // SIMD, from as many tiles and chunks as wavefronts up to three tiles each, one and a half from 33 heads on (attention
      // calls, four together over one alone, by tiles a SIMD, 8, 16 and 32 heads: 0.7 1.00 to 1.09; 1 to 2.9 0.91 to 0.95,
      // 3-bit keys 0.94 to 1.02; 3.4 0.98 to 1.05; 3.9 and more 0.99 to 1.12; 64 heads 1.3 0.97, 2.8 1.08; 4 and 3 bits 1 to
      // 1.2 0.96 to 0.98, 2 and more 1.01 to 1.10), and a compute unit for each (24 heads x 6k, 264 work-groups, 1.14).
      const int most_a_cu = kb + vb > 5 ? 0 : 8 * BH <= cus ? 12 : 4 * BH <= cus ? 6 : 0;
      waves = r > 4 && few_tiles && n_tiles + n_win_chunks >= per_head && BH * n_tiles <= most_a_cu * cus && BH * ceil_div(n_splits, 4) <= cus ? 4 : 1;
    }
    // Token counts on the device: the wavefronts planned for sequences of the bound's length go to the sequences by
    // their lengths, as many to one as it has partial slots, where there is something to gain: 16 sequences of 1k to
    // 16k tokens, 35.3 us per step with the same number each, 29.9 shared.  The sharing itself costs 1 to 1.7 us in
    // front of the first load, and packs the wavefronts of short sequences onto fewer compute units, so it wants
    // several tiles per wavefront (8 sequences x 8 heads, bound 2000 tokens: 13.8 against 14.9 shared; 8000 tokens,
    // lengths spread 16-fold: 18.2 against 15.9) and several wavefronts per head (16 x 32 heads, bound 4000: 28.8 against 38.2).
    // (Work-groups of one wavefront: 20 heads x 25k tokens 21.9 us, of two 24.3.)
    const long long shared = (long long)n_splits * c.batch;
    if (ragged && c.batch > 1 && c.batch <= kSharedBatchMost && (n_win_chunks + 1) * c.batch <= shared && n_tiles >= 6 * per_head && per_head >= 10) {
      shared_groups = (int)shared;
      n_splits = split_cap(c);
    }
  } else if (n_both > 0) {
    const long long blocks_per_split = (long long)c.batch * c.n_kv_heads * ceil_div(r, kHeadTile);
    long long s = ceil_div(2048, blocks_per_split);
    const long long by_len = ceil_div(n_both, 128);
    if (s > by_len) s = by_len;
    if (s > split_cap(c)) s = split_cap(c);
    if (s < 1) s = 1;
    n_splits = (int)s;
  }
  LaunchPlan p;
  p.n_splits = n_splits;
  p.n_win = (int)ceil_div(win_tokens, win_chunk_len);
  p.waves = waves;
  p.n_partials = joins ? n_partials : n_splits + p.n_win;
  p.shared_groups = shared_groups;
  p.joins = joins;
  const size_t partial_bytes = joins ? (size_t)kJoinBytes : (kHeadDim + 2) * sizeof(float);
  p.workspace_bytes = seq_bytes(c) + (size_t)c.batch * c.n_q_heads * (size_t)p.n_partials * partial_bytes + 64;
  return p;
}

}  // namespace innerq

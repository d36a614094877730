// Comparison kernel: fused split-K decode attention over an OUTER-dimension-grouped cache
// (kind = INNERQ_KIND_OUTER: keys grouped along tokens per channel, values along channels per
// token -- the layout the paper compares against, Figure "inner_outer" (a)).
//
// Same skeleton as the inner-grouped and fp16 kernels (one wavefront per token range, register prefetch of the next
// tile, window wavefronts in the same launch, same merge), and the stored fields go to the 16x16x32 fp16 matrix instructions
// as they are, masked in place (a field inside bits 0..10 of a 16-bit half reads as field * 2^position * 2^-24).  With outer
// grouping a group's scale depends on the index that is summed over, so it cannot be applied to the finished inner sum; it
// is folded into the OTHER operand instead:
//     q . K^[j]        = sum_c (q_c S_{c,T}) u[j][c]  +  sum_c q_c Zeff_{c,T}      (T: token group of j)
//     sum_j p_j V^[j][c] = sum_j (p_j S_{j,g}) u[j][c]  +  sum_j p_j Zeff_{j,g}    (g: channel group of c)
// (u = stored field, Zeff = Z for an asymmetric group and -2^(b-1) |S| for a symmetric one: Eq. hybrid_dequant.)
//
// The sixteen rows of a matrix instruction are what makes that cheap: four query heads times the (up to four) groups of a tile.
// A row (T, h) of the score product is q_h S_T, a column a half-word's worth of tokens; of the result, the rows of a column's own
// group are used.  So the folded operands are built in the registers that the instruction reads, 32 products a lane and tile, from
// scales that are loaded in that layout; the matrix cores have the room (one instruction in four would do for four heads).
//
// The packing runs ACROSS the inner dimension (a key word holds 16 tokens of ONE channel, a value word 16 channels of ONE
// token).  Sixteen columns of half-words that share a field position are what an instruction takes: a lane needs the same half-word
// of eight channels (tokens), which the transposing LDS read gives (ds_read_b64_tr_b16); one AND then makes two operand elements of
// two fields, and the instructions of one tile differ in the mask.  A tile is 16 half-words: 128 tokens of 2 bits, 64 of 4.
//
// What bounds it: vector issue (680 instructions to 112 matrix ones a tile of 2 bits, 282 of them the masks), at two wavefronts a
// SIMD, and in front of that the first tile's loads, which the whole chip asks for at once.  Time stamps, 8 x 8 heads x 8k tokens:
// first tile done at 9 us, 2.9 us each from then on, window chunks done at 7.4.  Attention calls (with the merge, in a graph), the
// kernel before this one, which took the folded operands through LDS to the 4x4x4 form (LDS busy 86 % of the time) -> now: 8 x 8
// heads, r = 4, 2 bits, 8k tokens 34.8 us -> 22.5, 32k 85.0 -> 50.7; 4 bits 8k 41.1 -> 26.4; 16 x 8 heads x 6k, r = 8, 103 -> 53; 8 heads x 8k 14.5 -> 11.0.
// A tile's loads go out as soon as the last one has left their registers (two sets of registers spilled, and a reload of a
// spilled value waits for every load in front of it: 32 us instead of 25 for the kernel alone).
#include "innerq_dev.h"
#include "window_pass.h"

namespace innerq {
namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

constexpr int D = kHeadDim;

// wave-wide maximum: the DPP form shared with the window pass
__device__ inline float wave_max_o(float x) { return window_wave_max(x); }

// A b-bit field masked in place inside a 16-bit half reads, as fp16, as field * 2^(bit position) * 2^-24 as long as it lies within
// bits 0..10 (the mantissa and the lowest exponent bit: the step from the denormals to the first binade keeps the spacing).  The
// matrix instruction aligns a denormal operand by the exponent 2^-14 and drops what falls off at the other end of its sum, so
// the fields are taken at positions 4 to 8 (4-bit: 2 and 6) from the word and two shifted copies (rms error of a sum of 32 products
// whose other factors span ten binades: position 0 1.5e-5, 4 5e-7, 6 6e-8).  f = index of the field inside its half.
template <int BITS>
struct InPlace {
  static constexpr int HALF = 16 / BITS;
  static constexpr int SHL = BITS == 2 ? 4 : 2, SHR = 6;
  static __host__ __device__ constexpr int from(int f) { return BITS == 2 ? (f < 2 ? 1 : f < 5 ? 0 : 2) : (f < 2 ? 1 : 2); }
  static __host__ __device__ constexpr int pos(int f) { return BITS * f + (from(f) == 1 ? SHL : from(f) == 2 ? -SHR : 0); }
  static __host__ __device__ constexpr uint32_t mask(int f) { return (uint32_t)(((1u << BITS) - 1u) * 0x00010001u) << pos(f); }
  // 2^24 / 2^(bit position): what brings the masked field back to its value
  static __host__ __device__ constexpr float undo(int f) { return (float)(1 << (24 - pos(f))); }
};

__device__ __forceinline__ half2_t as_half2(uint32_t w) { return __builtin_bit_cast(half2_t, w); }
__device__ __forceinline__ uint32_t as_u32(half2_t h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ half8_t as_half8(const u32x4& w) { return __builtin_bit_cast(half8_t, w); }
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }   // -126 <= e <= 127

// Least and largest of fp16 pairs, half by half, two pairs an instruction.
struct Range {
  uint32_t low = 0u, high = 0u;
  __device__ __forceinline__ void add(uint32_t a, uint32_t b) {
    asm("v_pk_minimum3_f16 %0, %1, %2, %0" : "+v"(low) : "v"(a), "v"(b));
    asm("v_pk_maximum3_f16 %0, %1, %2, %0" : "+v"(high) : "v"(a), "v"(b));
  }
  __device__ __forceinline__ uint32_t magnitudes() const {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, high & 0x7fff7fffu),
                                                                  __builtin_bit_cast(ushort2_t, low & 0x7fff7fffu)));
  }
};

// Power of two, as an fp16 pair, that brings the largest of the given fp16 magnitudes (bit patterns with
// the sign cleared, two per word; wave-wide) below 1, and its exponent: the scales of a tile are folded
// into the other operand of the products in that normalised form, so that the folded operands use the
// normal range of fp16 whatever the magnitude of the cache.
__device__ __forceinline__ int tile_shift(uint32_t magnitudes) {
  const uint32_t m = magnitudes & 0xffffu, n = magnitudes >> 16;
  const int top = (int)wave_max_o((float)(m > n ? m : n));       // (fp16 magnitudes order like integers)
  const int sh = 14 - (top >> 10);                                // value < 2^(biased exponent - 14)
  return sh < -14 ? -14 : sh;                                     // (at most 14: 2^sh is an fp16 number either way)
}
__device__ __forceinline__ half2_t pow2_half2(int e) {            // -14 <= e <= 15
  return as_half2((uint32_t)((15 + e) << 10) * 0x00010001u);
}

// The masked fields of position f of eight half-words (two a register), as one operand.
template <int BITS>
struct HalfWords {
  u32x4 w[3];
  __device__ __forceinline__ HalfWords(u32x2 lo, u32x2 hi) {
    w[0] = u32x4{lo.x, lo.y, hi.x, hi.y};
    w[1] = w[0] << InPlace<BITS>::SHL;
    w[2] = w[0] >> InPlace<BITS>::SHR;
  }
  __device__ __forceinline__ half8_t fields(int f) const { return as_half8(w[InPlace<BITS>::from(f)] & InPlace<BITS>::mask(f)); }
};

// Four 16-bit elements a lane from a 16 x 4 block of them per sixteen lanes: lane l passes the address of four elements and gets
// element l % 4 of what lanes l / 4, l / 4 + 4, + 8, + 12 of its sixteen address.
__device__ __forceinline__ u32x2 read_transposed(const unsigned char* p) {
  typedef __attribute__((address_space(3))) short4_t* lds_ptr;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)));
}

template <int BITS, int G>
struct Outer {
  static constexpr int HWT = 16 / BITS;                // tokens of a key half-word, channels of a value half-word
  static constexpr int TT = 16 * HWT;                  // tokens of a tile
  static constexpr int NT = TT / G;                    // token groups of a tile
  static constexpr int NG = D / G;                     // channel groups
  static constexpr int TPL = TT / 64;                  // tokens a lane takes through the softmax
  static constexpr int RUN = G * BITS / 8;             // bytes of one channel of a key group
  static constexpr int ROWB = D * BITS / 8;            // bytes of a value row
  static constexpr int KS = D / 32, VK = TT / 32;      // steps of 32 channels, of 32 tokens
  static constexpr int VS = D / (16 * HWT);            // sets of sixteen value half-words
  // LDS, bytes.  Key groups 64 bytes apart in the banks: a transposing read takes eight bytes of each of a channel's groups.
  static constexpr int KGROUP = 4096 / NT + 64, KEYS = NT * KGROUP, VALUES = TT * ROWB;
  static constexpr int SCORES = TT * 16;               // four heads
  static constexpr int ROW = TT * 2 + 64;              // a row of fp16 weights or scales: four rows and four steps of 16 bytes in different banks
  template <int NH4>
  static constexpr int bytes() { return KEYS + VALUES + SCORES + (4 * NH4 + 2 * NG) * ROW; }
};

// One tile as it is loaded.
template <int BITS, int G, bool ZK, bool ZV>
struct OuterRegs {
  using O = Outer<BITS, G>;
  u32x4 kc[4], vc[4];                                  // packed keys, values: 4 KB each, 16 bytes a lane and load, in memory order
  u32x4 ks[O::KS], kz[ZK ? O::KS : 1];                 // scales and zero-points of eight channels a step, of the lane's row's token group
  uint32_t vs[O::TPL][O::NG / 2], vz[O::TPL][O::NG / 2];   // fp16 pairs: channel groups of the lane's tokens
};

template <int BITS, int G, int NH4, bool ZK, bool ZV>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NH4 == 1 ? 2 : 1, 2)))
attention_outer_kernel(AttnArgs a, int n_both, int n_splits, WindowSet win) {
  using O = Outer<BITS, G>;
  using IP = InPlace<BITS>;
  using Regs = OuterRegs<BITS, G, ZK, ZV>;
  constexpr int NH = NH4 * 4, HWT = O::HWT, TT = O::TT, NT = O::NT, NG = O::NG, TPL = O::TPL;
  constexpr float kLevel = (float)(1 << (BITS - 1));   // symmetric zero-point: -2^(b-1) |S|  (Eq. hybrid_dequant)
  // A folded weight is a product rounded to fp16, and the field would multiply its error by up to 2^b - 1.  Taking the middle
  // of the field range out of the zero-point term with the ROUNDED products,  S u + Zeff = S (u - kMid) + (Zeff + kMid S),
  // leaves each one's error multiplied by |u - kMid| <= kMid only, and the explicit constant small.  (The folded queries have two
  // fp16 pieces, 2^-22 together, and their constant takes the exact Zeff.)
  constexpr float kMid = (float)((1 << BITS) - 1) * 0.5f;
  constexpr float kSlack = 6.0f;                       // scores may exceed the reference level by this (log2)

  const int lane = threadIdx.x;
  const long long bh = blockIdx.x;
  const int b = (int)(blockIdx.x / (uint32_t)a.n_kv_heads), hk = (int)(blockIdx.x % (uint32_t)a.n_kv_heads);
  const int r = a.n_q_heads / a.n_kv_heads;

  constexpr int kLdsBytes = O::template bytes<NH4>() > window_lds_bytes<NH4, G, true>() ? O::template bytes<NH4>() : window_lds_bytes<NH4, G, true>();
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLdsBytes];
  // (The grid is (sequence-heads, window chunks and then token ranges): ranges next to each other in it would meet on the same
  // dies where chunks and ranges together are a multiple of four or eight, 1024 heads x 4k tokens, 3 chunks and 1 range each, 331 us.)
  const int part = (int)(blockIdx.z * kGridParts + blockIdx.y);
  if (part >= win.n_chunks + n_splits) return;           // (a part that is not there: heads_by_parts)
  if (part < win.n_chunks) {
    WaveState<NH> st;
    window_pass<NH4, BITS, G, false, true, false>(a, bh, win.na, win.b0, win.nb, part, win.n_chunks, n_splits + part, lds, st, [] {});
    return;
  }
  const int n_tiles = (n_both + TT - 1) / TT;
  const int base_t = n_tiles / n_splits, rem_t = n_tiles % n_splits;
  const int s_idx = part - win.n_chunks;
  const int t0 = s_idx * base_t + (s_idx < rem_t ? s_idx : rem_t);
  const int t1 = t0 + base_t + (s_idx < rem_t ? 1 : 0);

  unsigned char* const keys = lds;
  unsigned char* const values = keys + O::KEYS;
  unsigned char* const scores = values + O::VALUES;
  unsigned char* const weights = scores + O::SCORES;                     // [NH] rows of softmax weights, then [NG] of scales, [NG] of constants
  unsigned char* const vscale = weights + NH * O::ROW;
  unsigned char* const vconst = vscale + NG * O::ROW;

  // Lane (quarter, col): as a row of the first operand, group block `rb` (of four) and head hl; as a column of the second and of
  // the result, half-word `col`; the result's rows in its four registers are the heads of group block `quarter`.
  const int quarter = lane >> 4, col = lane & 15, rb = col >> 2, hl = col & 3;
  const int row_T = rb * NT / 4, row_g = rb * NG / 4;
  const int col_T = col * NT / 16;                     // token group of the column's half-word

  const long long kgroups = a.capacity / G;
  const uint8_t* kcodes = a.k.codes + bh * kgroups * D * O::RUN;
  const __half* kscales = a.k.scales + bh * kgroups * D;
  const __half* kzeros = ZK ? a.k.zeros + bh * kgroups * D : nullptr;
  const uint8_t* vcodes = a.v.codes + bh * a.capacity * O::ROWB;
  const __half* vscales = a.v.scales + bh * a.capacity * NG;
  const __half* vzeros = ZV ? a.v.zeros + bh * a.capacity * NG : nullptr;
  const int last_row = n_both - 1, last_group = n_both / G - 1;        // (n_both: whole groups of tokens)
  const int tok0 = HWT * col + TPL * quarter;          // the lane's token(s) of a tile, from the softmax on
  float undo_k[TPL];                                   // of the field positions of their scores
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    undo_k[t] = IP::undo(t);
#pragma unroll
    for (int i = 1; i < 4; ++i) undo_k[t] = quarter == i ? IP::undo(TPL * i + t) : undo_k[t];
  }

  // Loads of a tile, each group of registers as soon as the previous tile has left it.  Groups and rows past the end re-read the
  // last ones (weight 0).  Behind the last tile every lane asks for the same bytes again: a load that is there on one of two
  // ways only would have everything before it waited for.  Offsets are 32-bit ones from a base in scalar registers.
  Regs cur;
  const uint32_t last_codes = (uint32_t)last_row * O::ROWB + (16 * lane) % O::ROWB;      // of the lane's 16-byte column of the value rows
  auto load_codes = [&](int tile, uint32_t lane16) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      constexpr int PER = 4 / NT;                       // loads of one token group
      int grp = tile * NT + x / PER;
      grp = grp > last_group ? last_group : grp;
      cur.kc[x] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kcodes + (uint32_t)(grp * (D * O::RUN) + (x % PER) * 1024 + lane16)));
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const uint32_t at = (uint32_t)tile * 4096u + 1024u * x + lane16;
      cur.vc[x] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vcodes + (at < last_codes ? at : last_codes)));
    }
  };
  auto load_key_scales = [&](int tile) {
    int grp = tile * NT + row_T;
    grp = grp > last_group ? last_group : grp;
    const uint32_t at = (uint32_t)(grp * D + 8 * quarter);
#pragma unroll
    for (int ks = 0; ks < O::KS; ++ks) cur.ks[ks] = *reinterpret_cast<const u32x4*>(kscales + at + 32 * ks);
    if constexpr (ZK) {
#pragma unroll
      for (int ks = 0; ks < O::KS; ++ks) cur.kz[ks] = *reinterpret_cast<const u32x4*>(kzeros + at + 32 * ks);
    }
  };
  auto load_value_scales = [&](int tile) {
    int row = tile * TT + tok0;
    row = row > last_row ? last_row + 1 - TPL : row;
    auto pairs = [&](const __half* p, uint32_t (&w)[TPL][NG / 2]) {
      constexpr int N = TPL * NG / 2;                   // 32-bit words
      const uint32_t* q = reinterpret_cast<const uint32_t*>(p + (uint32_t)(row * NG));
      uint32_t x[N];
      if constexpr (N == 4) { const u32x4 v = *reinterpret_cast<const u32x4*>(q); x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
      else if constexpr (N == 2) { const u32x2 v = *reinterpret_cast<const u32x2*>(q); x[0] = v.x; x[1] = v.y; }
      else x[0] = *q;
#pragma unroll
      for (int i = 0; i < N; ++i) w[i / (NG / 2)][i % (NG / 2)] = x[i];
    };
    pairs(vscales, cur.vs);
    if constexpr (ZV) pairs(vzeros, cur.vz);
  };

  {
    const int first = t0 < n_tiles ? t0 : n_tiles - 1;   // (a wavefront without a tile has something to read all the same)
    load_codes(first, 16u * lane);
    load_key_scales(first);
    load_value_scales(first);
  }

  // ---- query: the lane's eight channels a step of head hl, each head scaled by a power of two into [1/4, 1/2)
  u32x4 qn[NH4][O::KS];
  float qscale[NH];                                    // undoes that, log2(e) / sqrt(d) with it
#pragma unroll
  for (int n = 0; n < NH4; ++n) {
    const int h = 4 * n + hl;
    float q[O::KS][8], mx = 0.f;
#pragma unroll
    for (int ks = 0; ks < O::KS; ++ks) {
      u32x4 raw = {0u, 0u, 0u, 0u};
      if (h < r) raw = *reinterpret_cast<const u32x4*>(a.q + ((long long)b * a.n_q_heads + hk * r + h) * D + 32 * ks + 8 * quarter);
      const half8_t x = as_half8(raw);
#pragma unroll
      for (int e = 0; e < 8; ++e) q[ks][e] = (float)x[e];
      if (a.q_scale) {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[ks][e] = __half2float(scaled_half(q[ks][e], a.q_scale[hk * D + 32 * ks + 8 * quarter + e]));
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(q[ks][e]));
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const int e2 = mx > 0.f ? (int)((__float_as_uint(mx) >> 23) & 0xffu) - 127 + 2 : 0;
    const float f = pow2f(-e2);
#pragma unroll
    for (int ks = 0; ks < O::KS; ++ks) {
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = as_u32(half2_t{(_Float16)(q[ks][2 * i] * f), (_Float16)(q[ks][2 * i + 1] * f)});
      qn[n][ks] = u32x4{w[0], w[1], w[2], w[3]};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      qscale[4 * n + i] = 0.08838834764831845f * 1.4426950408889634f * pow2f(__builtin_amdgcn_readlane(e2, i));
  }

  // ---- running softmax state and accumulators.  m_run is a reference level that is raised (with a
  // wave-wide reduction and a rescale) only when a score exceeds it by more than kSlack.
  // oq[s][p][n]: channel p of the column's half-word of set s, the rows' heads 4 n .. 4 n + 3, in units of the masked fields and
  // of the running value shift (used where the row's channel group is the column's); oz: the constant terms; ol: the sum of the weights.
  float m_run[NH];
  float4_t oq[O::VS][HWT][NH4], oz[O::VS][NH4], ol[NH4];
  const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int h = 0; h < NH; ++h) m_run[h] = -INFINITY;
#pragma unroll
  for (int n = 0; n < NH4; ++n) {
    ol[n] = zero4;
#pragma unroll
    for (int s = 0; s < O::VS; ++s) {
      oz[s][n] = zero4;
#pragma unroll
      for (int p = 0; p < HWT; ++p) oq[s][p][n] = zero4;
    }
  }
  int shv_run = 64;                                    // the values' scales enter as S * 2^shv_run (64: nothing yet)
  const u32x4 ones_w = {0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u};
  const half8_t ones = as_half8(ones_w);
  const half8_t mids = ones * (half8_t)(_Float16)(-kMid);
  const half2_t level2 = {(_Float16)(-kLevel), (_Float16)(-kLevel)}, mid2 = {(_Float16)kMid, (_Float16)kMid}, zero2 = {(_Float16)0, (_Float16)0};
  // Place of token t in a row of weights or scales: of 32 tokens 16 x + 4 i + j, lane quarter i takes j = 0 .. 3 of both x (its
  // eight of a step; a transposing read of the value rows brings the four of one x, the quarters' rows next to each other).
  auto place = [](int t) { return (t & ~31) | ((t >> 2) & 3) << 3 | ((t >> 4) & 1) << 2 | (t & 3); };
  // value rows in LDS: at 4 bits, two steps of tokens in different halves of a 64-byte row
  auto value_at = [](int row, int byte) { return row * O::ROWB + (BITS == 2 ? byte : byte ^ (((row >> 2) & 1) << 5)); };

  for (int tile = t0; tile < t1; ++tile) {
    wave_fence();                                        // (the previous tile's reads are done)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      constexpr int PER = 4 / NT;
      *reinterpret_cast<u32x4*>(keys + (x / PER) * O::KGROUP + (x % PER) * 1024 + lane * 16) = cur.kc[x];
      *reinterpret_cast<u32x4*>(values + value_at((1024 * x + 16 * lane) / O::ROWB, (16 * lane) % O::ROWB)) = cur.vc[x];
    }
    wave_fence();
    const bool more = tile + 1 < t1;
    const int next_tile = more ? tile + 1 : tile;
    load_codes(next_tile, more ? 16u * lane : 0u);

    // ---- the powers of two that normalise the tile's scales
    Range krange, vrange;
#pragma unroll
    for (int ks = 0; ks < O::KS; ++ks) {
      krange.add(cur.ks[ks][0], cur.ks[ks][1]);
      krange.add(cur.ks[ks][2], cur.ks[ks][3]);
      if constexpr (ZK) {
        krange.add(cur.kz[ks][0], cur.kz[ks][1]);
        krange.add(cur.kz[ks][2], cur.kz[ks][3]);
      }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
      vrange.add(cur.vs[t][0], cur.vs[t][NG / 2 - 1]);
      if constexpr (ZV) vrange.add(cur.vz[t][0], cur.vz[t][NG / 2 - 1]);
    }
    const int shk = tile_shift(krange.magnitudes()), shv_tile = tile_shift(vrange.magnitudes());
    const half2_t fk = pow2_half2(shk);

    // ---- scores (Eq. att:1)
    float4_t su[HWT][NH4], sz[NH4];
#pragma unroll
    for (int n = 0; n < NH4; ++n) {
      sz[n] = zero4;
#pragma unroll
      for (int p = 0; p < HWT; ++p) su[p][n] = zero4;
    }
#pragma unroll
    for (int ks = 0; ks < O::KS; ++ks) {
      // channels 32 ks + 8 quarter + 4 x + j: a sixteen-lane read takes eight bytes (four half-words) of four channels
      const int c0 = 32 * ks + 8 * quarter + (col >> 2), chunk = col & 3, T = chunk * NT / 4;
      const unsigned char* at = keys + T * O::KGROUP + c0 * O::RUN + (chunk - T * 4 / NT) * 8;
      const HalfWords<BITS> w(read_transposed(at), read_transposed(at + 4 * O::RUN));
      u32x4 sw, zw;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // (the level meets the normalised scale: 2^(b-1) 2^shk by itself is no fp16 number where a tile's scales are tiny or zero)
        const half2_t signed_scale = as_half2(cur.ks[ks][i]) * fk;
        half2_t zn;
        if constexpr (ZK) {
          // the sign bit of a scale marks an asymmetric group, whose zero-point is stored; a symmetric
          // group stores +0 there and has Zeff = -2^(b-1) S
          zn = __builtin_elementwise_fma(as_half2(cur.kz[ks][i]), fk, __builtin_elementwise_max(signed_scale, zero2) * level2);
        } else {
          zn = signed_scale * level2;                    // (no flags: the scales are not negative)
        }
        sw[i] = as_u32(signed_scale) & 0x7fff7fffu;
        zw[i] = as_u32(zn);
      }
#pragma unroll
      for (int n = 0; n < NH4; ++n) {
        // q S in two fp16 pieces: with one, the rounding of a large channel's product (2^-12 of it, times
        // the field) shows in the output at 1e-3 on heavy-tailed keys
        u32x4 hw, lw;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const half2_t q2 = as_half2(qn[n][ks][i]), s2 = as_half2(sw[i]), hi = q2 * s2;
          const half2_t lo = __builtin_elementwise_fma(q2, s2, -hi);         // (the exact remainder, rounded once)
          hw[i] = as_u32(hi);
          lw[i] = as_u32(lo);
        }
        sz[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(qn[n][ks]), as_half8(zw), sz[n], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < HWT; p += 2) {               // (two chains in turn)
          const half8_t u0 = w.fields(p), u1 = w.fields(p + 1);
          su[p][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(hw), u0, su[p][n], 0, 0, 0);
          su[p + 1][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(hw), u1, su[p + 1][n], 0, 0, 0);
          su[p][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(lw), u0, su[p][n], 0, 0, 0);
          su[p + 1][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(lw), u1, su[p + 1][n], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    load_key_scales(next_tile);
    // ---- from the lanes whose rows are the column's group to one (two) tokens a lane, all heads
    float s[NH][TPL];
#pragma unroll
    for (int n = 0; n < NH4; ++n) {
      if (quarter * NT == col_T * 4) {
#pragma unroll
        for (int p = 0; p < HWT; ++p) {
          *reinterpret_cast<float4_t*>(scores + (16 * p + col) * 16) = su[p][n];
        }
      }
      wave_fence();
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        const float4_t v = *reinterpret_cast<const float4_t*>(scores + (16 * (TPL * quarter + t) + col) * 16);
#pragma unroll
        for (int h = 0; h < 4; ++h) s[4 * n + h][t] = __builtin_fmaf(v[h], undo_k[t], sz[n][h]) * (qscale[4 * n + h] * pow2f(-shk));
      }
      if (n + 1 < NH4) wave_fence();
    }
    // ---- running softmax (Eq. att:2); the weights are rounded to fp16 for the matrix cores and the
    // normaliser is the matrix cores' sum of the rounded weights
    if (tile * TT + TT - 1 > last_row) {                  // (uniform: the last tile, if it is not whole)
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        const bool valid = tile * TT + tok0 + t <= last_row;
#pragma unroll
        for (int h = 0; h < NH; ++h) s[h][t] = valid ? s[h][t] : -INFINITY;
      }
    }
    bool raise = false;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      float top = s[h][0];
      if constexpr (TPL == 2) top = fmaxf(top, s[h][1]);
      raise |= top > m_run[h] + kSlack;
    }
    const int shv_new = shv_tile < shv_run ? shv_tile : shv_run;
    if (__builtin_amdgcn_ballot_w64(raise) != 0 || shv_new != shv_run) {
      const float fshift = shv_run == 64 ? 0.f : pow2f(shv_new - shv_run);   // (nothing accumulated yet: any factor)
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        float top = s[h][0];
#pragma unroll
        for (int t = 1; t < TPL; ++t) top = fmaxf(top, s[h][t]);
        const float m_new = fmaxf(m_run[h], wave_max_o(top));
        const float alpha = __builtin_amdgcn_exp2f(m_run[h] - m_new);        // 0 the first time
        m_run[h] = m_new;
        ol[h / 4][h % 4] *= alpha;
#pragma unroll
        for (int x = 0; x < O::VS; ++x) {
          oz[x][h / 4][h % 4] *= alpha * fshift;
#pragma unroll
          for (int p = 0; p < HWT; ++p) oq[x][p][h / 4][h % 4] *= alpha * fshift;
        }
      }
      shv_run = shv_new;
    }
    {
      // sum_j p_j V^[j][c] = sum_j (p_j S_{j,g}) u[j][c] + sum_j p_j Zeff_{j,g}  (g = channel group of c):
      // the weights, the tokens' scales and their constants Zeff + kMid S, to where the operands' lanes read eight tokens each
      const half2_t fv = pow2_half2(shv_run);
      half2_t sn[TPL][NG / 2], zn[TPL][NG / 2];
#pragma unroll
      for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int i = 0; i < NG / 2; ++i) {
          sn[t][i] = as_half2(cur.vs[t][i] & 0x7fff7fffu) * fv;
          if constexpr (ZV) {
            const half2_t ssym = __builtin_elementwise_max(as_half2(cur.vs[t][i]), zero2) * fv;
            zn[t][i] = __builtin_elementwise_fma(as_half2(cur.vz[t][i]), fv, ssym * level2);
          } else {
            zn[t][i] = sn[t][i] * level2;
          }
          zn[t][i] = __builtin_elementwise_fma(sn[t][i], mid2, zn[t][i]);
        }
      const int at = place(tok0) * 2;
      auto put = [&](unsigned char* row, _Float16 x0, _Float16 x1) {
        if constexpr (TPL == 2) *reinterpret_cast<uint32_t*>(row + at) = as_u32(half2_t{x0, x1});
        else *reinterpret_cast<_Float16*>(row + at) = x0;
      };
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        put(vscale + g * O::ROW, sn[0][g / 2][g & 1], sn[TPL - 1][g / 2][g & 1]);
        put(vconst + g * O::ROW, zn[0][g / 2][g & 1], zn[TPL - 1][g / 2][g & 1]);
      }
#pragma unroll
      for (int h = 0; h < NH; ++h)
        put(weights + h * O::ROW, (_Float16)__builtin_amdgcn_exp2f(s[h][0] - m_run[h]), (_Float16)__builtin_amdgcn_exp2f(s[h][TPL - 1] - m_run[h]));
    }
    load_value_scales(next_tile);
    wave_fence();
    // ---- values (Eq. att:3)
#pragma unroll
    for (int ks = 0; ks < O::VK; ++ks) {
      const int at = 64 * ks + 16 * quarter;
      const u32x4 sw = *reinterpret_cast<const u32x4*>(vscale + row_g * O::ROW + at);
      half8_t pw[NH4], aw[NH4];
#pragma unroll
      for (int n = 0; n < NH4; ++n) {
        pw[n] = *reinterpret_cast<const half8_t*>(weights + (4 * n + hl) * O::ROW + at);
        aw[n] = pw[n] * as_half8(sw);
        ol[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pw[n], ones, ol[n], 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < O::VS; ++x) {
        const int row = 32 * ks + 4 * quarter + (col >> 2), byte = 32 * x + 8 * (col & 3);
        const HalfWords<BITS> w(read_transposed(values + value_at(row, byte)), read_transposed(values + value_at(row + 16, byte)));
        const half8_t zw = *reinterpret_cast<const half8_t*>(vconst + ((16 * x + col) * HWT / G) * O::ROW + at);
#pragma unroll
        for (int n = 0; n < NH4; ++n) {
          oz[x][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pw[n], zw, oz[x][n], 0, 0, 0);
          oz[x][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aw[n], mids, oz[x][n], 0, 0, 0);       // - kMid * (weights times scales, as rounded)
#pragma unroll
          for (int p = 0; p < HWT; ++p) oq[x][p][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aw[n], w.fields(p), oq[x][p][n], 0, 0, 0);
        }
      }
    }
  }

  // ---- partial result: undo the field positions and the value shift, add the constant term
  const float fv_undo = shv_run == 64 ? 0.f : pow2f(-shv_run);
  const int slot = s_idx;
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    if (h < r) {
      const long long bhq = (long long)b * a.n_q_heads + hk * r + h;
#pragma unroll
      for (int x = 0; x < O::VS; ++x) {
        if (quarter * NG == ((16 * x + col) * HWT / G) * 4) {
          float* dst = &a.ws_o[(bhq * a.n_partials + slot) * D + (16 * x + col) * HWT];
#pragma unroll
          for (int p = 0; p < HWT; p += 4) {
            float4_t o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(oq[x][p + i][h / 4][h % 4], IP::undo(p + i), oz[x][h / 4][h % 4]) * fv_undo;
            *reinterpret_cast<float4_t*>(dst + p) = o;
          }
        }
      }
      if (lane == 0) {
        a.ws_ml[(bhq * a.n_partials + slot) * 2 + 0] = m_run[h] * 0.6931471805599453f;
        a.ws_ml[(bhq * a.n_partials + slot) * 2 + 1] = ol[h / 4][h % 4];
      }
    }
  }
}

template <int BITS, int G, bool ZK, bool ZV>
hipError_t launch_z(const AttnArgs& a, int n_both, int n_splits, const WindowSet& win, const Launch& L) {
  const int r = a.n_q_heads / a.n_kv_heads;
  const HeadsByParts g = heads_by_parts((long long)a.batch * a.n_kv_heads, (long long)n_splits + win.n_chunks);
  const dim3 grid(g.x, g.y, g.z);
  if (r <= 4)
    hipExtLaunchKernelGGL((attention_outer_kernel<BITS, G, 1, ZK, ZV>), grid, dim3(64), 0, L.stream, L.ev_start,
                          L.ev_stop, 0, a, n_both, n_splits, win);
  else
    hipExtLaunchKernelGGL((attention_outer_kernel<BITS, G, 2, ZK, ZV>), grid, dim3(64), 0, L.stream, L.ev_start,
                          L.ev_stop, 0, a, n_both, n_splits, win);
  return hipGetLastError();
}

template <int BITS, int G>
hipError_t launch_t(const AttnArgs& a, int n_both, int n_splits, const WindowSet& win, const Launch& L) {
  const bool zk = a.k.zeros != nullptr, zv = a.v.zeros != nullptr;
  if (zk && zv) return launch_z<BITS, G, true, true>(a, n_both, n_splits, win, L);
  if (zk) return launch_z<BITS, G, true, false>(a, n_both, n_splits, win, L);
  if (zv) return launch_z<BITS, G, false, true>(a, n_both, n_splits, win, L);
  return launch_z<BITS, G, false, false>(a, n_both, n_splits, win, L);
}

}  // namespace

bool attention_outer_supported(const AttnArgs& a) {
  const int r = a.n_q_heads / a.n_kv_heads;
  return a.k.form == kPerChannel && a.v.form == kPerToken && (a.bits == 2 || a.bits == 4) && a.v_bits == a.bits && r <= 8 &&
         a.capacity * D <= (1LL << 31) && !a.pages.table;
}

namespace {
// Resident workgroups per compute unit of one instance: the runtime's answer, bounded by the LDS the
// instance declares rounded up to the allocation granule (the runtime's answer has been one too many for a
// workgroup of 27 264 bytes: six counted, five resident, and the launch ran in two rounds).
template <int BITS, int G, int NH4>
int resident_outer() {
  const auto kernel = attention_outer_kernel<BITS, G, NH4, true, true>;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, 64, 0) != hipSuccess || n <= 0) return 4;
  hipFuncAttributes fa;
  if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel)) == hipSuccess && fa.sharedSizeBytes > 0) {
    const size_t granule = 1024, lds_per_cu = 160 * 1024;
    const int by_lds = (int)(lds_per_cu / (((fa.sharedSizeBytes + granule - 1) / granule) * granule));
    if (by_lds >= 1 && by_lds < n) n = by_lds;
  }
  return n;
}
}  // namespace

int attention_outer_tile_tokens(const AttnArgs& a) { return a.bits == 2 ? Outer<2, 32>::TT : Outer<4, 32>::TT; }

int attention_outer_waves_per_cu(const AttnArgs& a) {
  // 64-thread groups: registers decide (two wavefronts a SIMD; one with more than four heads per kv head)
  static CachedInt c[2][2][2];
  const int r = a.n_q_heads / a.n_kv_heads;
  const bool b4 = a.bits == 4, g64 = a.group == 64, wide = r > 4;
  return c[b4][g64][wide].get([&] {
    if (b4) {
      if (g64) return wide ? resident_outer<4, 64, 2>() : resident_outer<4, 64, 1>();
      return wide ? resident_outer<4, 32, 2>() : resident_outer<4, 32, 1>();
    }
    if (g64) return wide ? resident_outer<2, 64, 2>() : resident_outer<2, 64, 1>();
    return wide ? resident_outer<2, 32, 2>() : resident_outer<2, 32, 1>();
  });
}

hipError_t launch_attention_outer(const AttnArgs& a, long long n_both_ll, int n_splits, const WindowSet& win,
                                  hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int n_both = (int)n_both_ll;
  const Launch L = {stream, ev_start, ev_stop};
  if (a.bits == 2 && a.group == 32) return launch_t<2, 32>(a, n_both, n_splits, win, L);
  if (a.bits == 2 && a.group == 64) return launch_t<2, 64>(a, n_both, n_splits, win, L);
  if (a.bits == 4 && a.group == 32) return launch_t<4, 32>(a, n_both, n_splits, win, L);
  if (a.bits == 4 && a.group == 64) return launch_t<4, 64>(a, n_both, n_splits, win, L);
  return hipErrorInvalidValue;
}

}  // namespace innerq

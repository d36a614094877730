// Fused dequantise + score + softmax + value kernel for the inner-grouped cache
// (keys per-token group-wise, values per-channel group-wise; Section "InnerQ").
//
// One wavefront streams a contiguous range of quantised tokens once and serves
// every query head that shares the kv head from those bytes.
//
// Why the grouping matters here (Section "InnerQ", Figure "inner_outer"): with
// groups along the inner dimension of each product, a group's scale and
// zero-point factor out of the inner sum,
//     q . k_j      = sum_g |S_jg| * (sum_{c in g} q_c u_jc) + Zeff_jg * (sum_{c in g} q_c)
//     sum_j p_j v_jc = sum_T |S_Tc| * (sum_{j in T} p_j u_jc) + Zeff_Tc * (sum_{j in T} p_j)
// (u = stored field, Zeff = Z for an asymmetric group and -|S| 2^(b-1) for a
// symmetric one: Eq. hybrid_dequant), so the inner sums run on the raw integer
// fields and one multiply per group applies the scale.
//
// Mapping to CDNA4:
//   * inner sums run on the matrix cores with v_mfma_f32_16x16x32_f16 as four 4 x 8 x 16 products side by side: the
//     A operand (4 query heads x 8 inner indices) stands on the diagonal of 16 x 32, and lane l's four results are its
//     own column (8 inner indices of its token or channel) for the four heads.  In the score pass a lane owns one
//     token, in the value pass two channels, and the result lands in the lane that holds that token's / channel's
//     scale: no cross-lane traffic.  (The 4x4x4 form has the same multiply rate at twice the instructions; a tile
//     takes 36 instead of 82, since the normaliser needs one with all A rows alike instead of a chain.)
//   * a b-bit field becomes an fp16 operand with ONE and per two fields: masked in
//     place inside a 16-bit half it is an fp16 denormal u * 2^(off - 24) (the matrix cores keep fp16
//     denormals; see Fields for the offsets); the offset's factor is folded into
//     the A operand (query / probabilities), the constant into the group scale.
//     Measured, 8 x 8 heads x 32k tokens, 2-bit, step: 41.2 us -> 39.8 (3-bit 59.3 -> 56.9; 8 query heads per kv head,
//     16k tokens, 3-bit keys 31.7 -> 27.5; sequences of 1k to 16k tokens 39.3 -> 36.6), error against fp64 2.8e-4 -> 2.3e-4
//     (4-bit, 4k tokens 5.4e-4 -> 2.7e-4; 128k tokens 2.5e-4 -> 1.2e-4; eight heads, 16k tokens 1.8e-4 -> 1.1e-4).
//   * 3-bit fields are stored as a plane of 2-bit low parts followed by a plane of
//     high bits; the high bits are 1-bit fields of the same kind (2^(pos - 24)) and
//     join the same MFMA chains through operand tables that carry their weight 4.
//     Keys and values may have different widths (template parameters KB, VB).
//   * softmax probabilities are rounded to fp16 for the value pass and the
//     normaliser is the MFMA sum of those same rounded values (an extra all-ones B
//     operand), so the weights stay consistent.
//   * schedule: n_splits wavefronts per (batch, kv-head), all resident at once at two per SIMD, by themselves or (launches that
//     join, some with eight heads) in work-groups of up to eight that share the query tables; contiguous tile ranges; two
//     register buffers in ping-pong; the wavefront that is behind its SIMD partner gets the higher issue priority, so both
//     finish together.
//   * one launch, where the plan (plan.h) says so: a work-group's wavefronts meet in LDS at the end, the work-groups of a (batch,
//     kv-head) through the workspace (merge.h), and the append of a decode step's token is taken by the first wavefront
//     that is through.  A launch for merge and append behind this one takes 3.4 us after a short kernel and 4.7 after a
//     long one, whatever it does.  Per step, with the merge -> joined: 1 head x 512 tokens 11.8 us -> 9.0, 32 heads x 4k
//     12.8 -> 11.6, 8 x 8 x 32k 40.0 -> 37.9, 32 x 8 x 8k 41.8 -> 38.7, 4 x 8 x 128k 72.7 -> 70.3, 3-bit 8 x 8 x 32k 56.9 -> 54.6.
//   * paged store: this file is compiled for both stores, for launches that join and for those that do not (and, to build in
//     parallel, for both group sizes).  attention_inner_paged*.hip include it with INNERQ_PAGED_STORE set and get the kernels
//     that look every tile up in the page table (a page is one 64-token tile); the builds for the contiguous store carry no
//     trace of that.  attention_join*.hip get the kernels that join and append, compiled with NaN honoured, as the quantiser
//     wants it; the others need no NaN canonicalisation around their maxima.
#include "innerq_dev.h"
#ifndef INNERQ_INNER_LAUNCH
#define INNERQ_PAGED_STORE 0
#define INNERQ_INNER_JOIN 0
#define INNERQ_INNER_LAUNCH launch_inner_g32
#define INNERQ_INNER_GROUP 32
#endif
#if INNERQ_INNER_JOIN
#define INNERQ_CONTRACTED
#include "quantize_rows.h"
#endif
#include "window_pass.h"
#include "merge.h"

namespace innerq {
namespace {

constexpr bool kPagedStore = INNERQ_PAGED_STORE != 0;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int D = kHeadDim;
constexpr int TILE = 64;                       // tokens per wave iteration (one per lane)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSmScale = 0.08838834764831845f;   // 1/sqrt(128)

// Half `hi` (0 or 1) of a 32-bit word as fp16.
__device__ inline _Float16 half_of(uint32_t w, int hi) {
  return __builtin_bit_cast(_Float16, (unsigned short)(hi ? (w >> 16) : (w & 0xffffu)));
}

// max(x, 0), half by half, in one instruction (the compiler would put another before it for signalling NaNs).
__device__ __forceinline__ half2_t positive_part(half2_t x) {
  half2_t y;
  asm("v_pk_max_f16 %0, %1, 0" : "=v"(y) : "v"(x));
  return y;
}

// Where the fields of a 32-bit word are masked out: after an optional shift of the whole word, field f of a 16-bit
// half sits at bit off(f) of it.  The offsets are kept high in the 10 mantissa bits: the matrix cores line products
// up by the operands' exponent fields, and a denormal's is that of 2^-14 however many leading zeros it has, so a
// field at offset 0 loses about ten bits of its product's sum (measured: 1e-6 relative, rounded towards zero,
// with the fields of a word at offsets 0 .. 8; nothing lost with the offsets below).
template <int BITS>
struct Fields {
  static constexpr int FPW = 32 / BITS;        // fields per 32-bit word
  static constexpr int HALF = FPW / 2;         // fields per 16-bit half
  static constexpr int MPW = HALF / 2;         // groups of two field positions x two halves (two groups a matrix instruction)
  // shift of the word that field position f is read from: 0, 1 (left by SHL) or 2 (right by SHR)
  static constexpr int SHL = BITS == 2 ? 4 : BITS == 4 ? 2 : 8;
  static constexpr int SHR = BITS == 1 ? 8 : 6;
  static __host__ __device__ constexpr int from(int f) {
    return BITS == 2 ? (f < 2 ? 1 : f < 5 ? 0 : 2) : BITS == 4 ? (f < 2 ? 1 : 2) : (f < 2 ? 1 : f < 10 ? 0 : 2);
  }
  static __host__ __device__ constexpr int off(int f) { return BITS * f + (from(f) == 1 ? SHL : from(f) == 2 ? -SHR : 0); }
  static __host__ __device__ constexpr uint32_t mask(int f) {
    return (uint32_t)(((1u << BITS) - 1u) * 0x00010001u) << off(f);
  }
  static __host__ __device__ constexpr uint32_t ones(int f) { return 0x00010001u << off(f); }
  // index of inner position e (0..FPW) inside its word's operand table: [mfma][slot]
  static __host__ __device__ constexpr int slot(int e) {
    const int hi = e / HALF, f = e % HALF;
    return (f / 2) * 4 + (f % 2) * 2 + hi;
  }
};

// A word and its two shifted copies.
template <int BITS>
struct Shifted {
  uint32_t w[3];
  __device__ __forceinline__ explicit Shifted(uint32_t v) {
    w[0] = v;
    w[1] = v << Fields<BITS>::SHL;
    w[2] = v >> Fields<BITS>::SHR;
  }
  __device__ __forceinline__ Shifted() {}
};

// B operand of one matrix instruction: the fields of positions 2 m .. 2 m + 3 of both halves (m even).
template <int BITS>
__device__ inline half8_t operand(const Shifted<BITS>& w, int m) {
  using F = Fields<BITS>;
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = 2 * m + i;
    r[i] = w.w[F::from(f)] & F::mask(f);
  }
  return __builtin_bit_cast(half8_t, u32x4{r[0], r[1], r[2], r[3]});
}

// 1 in the place of every field: eight consecutive entries of an operand table, from entry 8 kb on.
template <int BITS>
__device__ inline half8_t ones_operand(int kb) {
  using F = Fields<BITS>;
  constexpr int PER = F::FPW / 8;              // eights per word
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = F::ones(i);
#pragma unroll
    for (int e = 1; e < PER; ++e) r[i] = kb % PER == e ? F::ones(4 * e + i) : r[i];
  }
  return __builtin_bit_cast(half8_t, u32x4{r[0], r[1], r[2], r[3]});
}

__device__ inline float wave_max(float x) {
  // butterflies inside a row of 16 lanes via DPP, then the four rows through scalar registers
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true)));
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true)));
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true)));
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true)));
  const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 0));
  const float b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 16));
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 32));
  const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

// Maximum over the lanes of the same row parity (rows of 16 lanes).
__device__ inline float parity_max(float x, int par) {
  x = fmaxf(x, lane_moved<0xB1>(x));
  x = fmaxf(x, lane_moved<0x4E>(x));
  x = fmaxf(x, lane_moved<0x141>(x));
  x = fmaxf(x, lane_moved<0x140>(x));
  const float even = fmaxf(from_lane(x, 0), from_lane(x, 32)), odd = fmaxf(from_lane(x, 16), from_lane(x, 48));
  return par ? odd : even;
}

// Inclusive sums over the lanes.
struct Scan { int upto, total; };
__device__ inline Scan wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);     // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);     // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);     // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);     // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2, 3
  return {x, __builtin_amdgcn_readlane(x, 63)};
}

template <typename T>
__device__ inline T stream_load(const T* p) { return __builtin_nontemporal_load(p); }

// Everything one wave iteration reads from the quantised store.  3-bit codes are two planes per
// packed run (2-bit low parts, then 1-bit high parts): a key row is 32 + 16 bytes, one channel of
// one value group G/4 + G/8 bytes.
template <int KB, int VB, int G>
struct TileRegs {
  static constexpr int KC = D * KB / 8 / 16;           // 16-byte pieces of one key row
  static constexpr int NG = D / G;                     // key groups per token
  static constexpr int GPT = TILE / G;                 // value token-groups per tile
  static constexpr int CW = G * VB / 32;               // words of one channel of one value group
  static constexpr int VW = 2 * CW;                    // ... of this lane's two channels
  u32x4 kc[KC];
  uint32_t ks[NG / 2], kz[NG / 2];                     // fp16 pairs
  uint32_t vw[GPT][VW];
  uint32_t vs[GPT], vz[GPT];                           // fp16 pairs (this lane's two channels)
  long long gshift;                                    // paged store: where the tile's value groups sit (wave-uniform)
  __device__ uint32_t k_word(int w) const { return kc[w / 4][w % 4]; }                 // (low) plane of the row
  __device__ uint32_t k_high(int w) const { return kc[(D * 2 / 32 + w) / 4][(D * 2 / 32 + w) % 4]; }
  __device__ uint32_t v_word(int gi, int ch, int w) const { return vw[gi][ch * CW + w]; }
  __device__ uint32_t v_high(int gi, int ch, int w) const { return vw[gi][ch * CW + G * 2 / 32 + w]; }
};

// Tiles' worth of time a window chunk of `len` tokens costs the wavefront that carries it.  The
// chunk runs at the lowest issue priority next to a partner that is busy about three quarters of
// the time, so its wall time is several times its own instruction count; the slope is the one that
// balances the launch best when swept (3 to 11 per 64 tokens: flat between 5 and 11 on the 32k-token
// G = 32 configuration, best at 9; best at 5 on the 8k x 32 G = 64 one, 6 % better than at 11).
__host__ __device__ inline int window_cost(long long len, int group) { return (int)(2 + (group == 64 ? 5 : 9) * len / 64); }

// LDS of a work-group, in bytes: what its wavefronts share, then OWN for each.
template <int KB, int VB, int G, int NH4>
struct Lds {
  static constexpr int NH = 4 * NH4, NG = D / G;
  static constexpr int QS = D + 8, PS = TILE + 8;                  // a head's row of the query / probability tables (halves)
  static constexpr int ZEROS = QS;                                 // a row of zeros
  static constexpr int QSUM = (NH * QS * (KB == 3 ? 2 : 1) + ZEROS) * 2;
  static constexpr int COEF = QSUM + NH4 * NG * 4 * 4;
  static constexpr int COUNT = COEF + NH * 4;                      // wavefronts that have come to the end
  static constexpr int SHARED = COUNT + 16;
  static constexpr int most(int x, int y) { return x > y ? x : y; }
  static constexpr int OWN = most(most(NH * PS * 2 * (VB == 3 ? 2 : 1), window_lds_bytes<NH4, G, false>()), NH * (D + 2) * 4);
  static_assert(QSUM % 16 == 0 && SHARED % 16 == 0 && OWN % 16 == 0, "16-byte pieces");
  static constexpr int bytes(int waves) { return SHARED + waves * OWN; }
};

// KB, VB: widths of the key and value codes.  ZK: the key zero-point array exists (the key mode is not
// symmetric-only).  ZV: 0 = no value zero-point array; 1 = zero-points read densely, one tile ahead with
// everything else; 2 = sparse (Section "Sparsity of M": the flag matrix is mostly zero): a lane reads the
// zero-points of its two channels only if one of the two groups is flagged asymmetric (the flag is the
// sign bit of the scale it already holds), at the start of the tile that needs them, so a 128-byte line
// of zero-points (64 channels of one token-group) that holds no asymmetric group is never fetched.
// JOIN: the launch joins its own partial results and may append a step's token; else it leaves them to the merge, and the token
// counts may live on the device.  (One kernel for both had worse code in the tile loop: 3-bit keys, 8 x 8 heads x 8k tokens,
// attention call 19.7 us before, 21.1, 19.9 with the two apart.)
constexpr bool JOIN = INNERQ_INNER_JOIN != 0;
// (a launch that cannot append has no use for its arguments)
#if INNERQ_INNER_JOIN
typedef QuantArgs AppendArgs;
#else
typedef int AppendArgs;
#endif

// ALONE: one wavefront a work-group, as most launches are that leave their partials to the merge.  It shares nothing: no
// barrier, no second copy of the query set-up, constants of the heads straight from lane to lane, and a wavefront without a
// tile has no tables.  (Against kernels for any number of wavefronts, us: 16 paged sequences of 1k to 16k tokens 28.4 -> 27.8;
// attention calls, eight query heads per kv head, 4 x 8 x 16k, 3-bit keys 25.6 -> 23.5, 8 heads x 0.9k at 4 bits 12.4 -> 11.6.)
template <int KB, int VB, int G, int NH4, bool ZK, int ZV, bool ALONE>
__global__ void __launch_bounds__(ALONE ? 64 : 512) __attribute__((amdgpu_waves_per_eu(2, 2))) attention_inner_kernel(AttnArgs a_in, int n_both_in, int n_splits, WindowSet win_in, int win_tiles_in, int base_t_in,
                                                                                                 int rem_t_in, int r, int waves_in, int groups_in, int appends, AppendArgs append) {
  constexpr int LBK = KB == 3 ? 2 : KB, LBV = VB == 3 ? 2 : VB;   // field width of the (low) plane
  constexpr bool HIK = KB == 3, HIV = VB == 3;                     // a plane of high bits follows it
  using FK = Fields<LBK>;
  using FV = Fields<LBV>;
  using F1 = Fields<1>;
  using Regs = TileRegs<KB, VB, G>;
  constexpr int NG = Regs::NG, GPT = Regs::GPT, KC = Regs::KC, VW = Regs::VW;
  constexpr int HWG = G / 32;                          // words of the high-bit plane per group
  constexpr int NW = D / FK::FPW;                      // words per key row
  constexpr int WPGK = G / FK::FPW, WPGV = G / FV::FPW;   // words per group (key: channels; value: tokens)
  constexpr int MPWK = FK::MPW, MPWV = FV::MPW;
  constexpr int HALFK = 1 << (KB - 1), HALFV = 1 << (VB - 1);
  // A field of value u at offset `off` is the fp16 number u 2^(off - 24); the table entries of the other operand carry
  // 2^(CK - off) (queries) and 2^(CV - off) (probabilities), 4 times that in the plane of high bits.  CK, CV: as large
  // as fp16 allows with queries below 2^9, probabilities up to 2^kSlack and offsets from 4 (2-bit) or 2 on.
  constexpr int CK = KB == 2 ? 10 : KB == 4 ? 8 : 6, CV = VB == 2 ? 13 : VB == 4 ? 11 : 10;
  constexpr int NH = NH4 * 4;
  constexpr int CH = NH4;                              // chains of matrix instructions, each over 64 / CH of the columns
  // Field positions of a 16-bit half of a high plane's word that one lane takes (eight heads and groups of 32: a word is a
  // whole group's, and two lanes share it).
  constexpr int F1PER = NH4 == 2 && G == 32 ? 8 : 16;

  // No division on the way to the first load: the grid is (splits, kv heads, batch), and the
  // host passes the quotients (heads per kv head; tiles per plain wavefront and their remainder).
  const int lane = threadIdx.x & 63;
  const int waves = ALONE ? 1 : waves_in;
  const int wave = ALONE ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // (waves, groups: of a work-group / launch, as arguments: the built-in sizes are loads of their own)
  const int hk = (int)blockIdx.y;
  int b = (int)blockIdx.z, group = (int)blockIdx.x;      // sequence; work-group of its (b, hk)
  const int n_groups = groups_in;
  // The host's plan holds for every sequence -- unless the token counts live on the device
  // (a.n_dev: one count per sequence, the tokens cached BEFORE this step; attention runs over them
  // plus the new token).  Then the launch shape and the window chunks are the
  // host's, planned for the longest sequence allowed, and everything that depends on the length is
  // recomputed here for this wavefront's sequence: the partition of Eq. kv_cache_init_quantized_window,
  // the window set and the split of the tiles over the wavefronts.  With shared_groups (BALANCED below) the wavefronts
  // of a kv head are shared out over the sequences by their lengths; n_splits is then the most one sequence may get
  // (its partial slots).  Wavefronts left without a tile write an empty partial, or nothing beyond their sequences.
  AttnArgs a = a_in;
  int n_both = n_both_in, win_tiles = win_tiles_in, base_t = base_t_in, rem_t = rem_t_in;
  WindowSet win = win_in;
  if (ALONE && a_in.n_dev) {
    const int w_recent = a.k.slots - 1;                  // (the per-token key ring has w_recent + 1 slots)
    const int n_chunks = win.n_chunks;
    // counts fit 24 bits (capacity * head_dim <= 2^31); outside their bounds they are clamped
    auto clamped = [&](int n) { return n + 1 < 1 ? 1 : ((long long)n + 1 > a.capacity ? (int)a.capacity : n + 1); };
    struct Length { int n, n_sink, vq, win, tiles, cost; };
    auto length = [&](int n) -> Length {
      Length x;
      x.n = n;
      x.n_sink = n < a.w_sink ? n : a.w_sink;
      int mid = n - a.w_sink - w_recent;
      mid = mid < 0 ? 0 : mid;
      x.vq = mid - mid % G;
      const int b0 = a.w_sink + x.vq;
      x.win = x.n_sink + (n > b0 ? n - b0 : 0);
      x.tiles = (x.vq + TILE - 1) / TILE;
      x.cost = n_chunks > 0 ? window_cost((uint32_t)(x.win + n_chunks - 1) / (uint32_t)n_chunks, G) : 0;
      return x;
    };
    int n;
    if (a.shared_groups > 0) {
      // BALANCED (a sequence a lane): a number of tiles per wavefront, window chunks counted in tiles, with which the
      // sequences' wavefronts fit the launch: the smallest one below 8, at most an eighth above it beyond (every try is a
      // scan of the lengths, in front of the first load).  No fewer than four tiles (a wavefront pays its query set-up
      // once).
      const int total = groups_in;
      const int n_lane = clamped(lane < a.batch ? a_in.n_dev[lane] : 0);
      const Length x = length(n_lane);
      const int work = lane < a.batch ? x.tiles + n_chunks * x.cost : 0;
      int quota = (wave_scan(work).total + total - 1) / total;
      quota = quota < 4 ? 4 : quota;
      int mine;
      Scan sc;
      for (;;) {
        mine = (work + quota - 1) / quota;
        mine = mine < n_chunks + 1 ? n_chunks + 1 : mine;
        mine = mine > n_splits ? n_splits : mine;
        mine = lane < a.batch ? mine : 0;
        sc = wave_scan(mine);
        if (sc.total <= total) break;                    // (the host: batch * (n_chunks + 1) <= total)
        quota += 1 + (quota >> 3);
      }
      b = __popcll(__builtin_amdgcn_ballot_w64(lane < a.batch && group >= sc.upto));
      if (b >= a.batch) return;                            // (wave-uniform)
      n_splits = __builtin_amdgcn_readlane(mine, b);
      group -= __builtin_amdgcn_readlane(sc.upto, b) - n_splits;
      n = __builtin_amdgcn_readlane(n_lane, b);            // (not read again: a memory round trip)
    } else {
      n = clamped(a_in.n_dev[b]);
    }
    const Length x = length(n);
    if (group == 0 && hk == 0 && lane == 0) {
      if (a.n_copy) a.n_copy[b] = x.n - 1;                 // for the append that follows
      if (a.n_valid) a.n_valid[b] = n_splits + n_chunks;   // partial results of this sequence's heads
    }
    a.n_tokens = x.n;
    a.k.n_sink = x.n_sink; a.v.n_sink = x.n_sink;
    a.k.n_quant = x.n - a.w_sink - w_recent > 0 ? x.n - a.w_sink - w_recent : 0;
    a.v.n_quant = x.vq;
    n_both = x.vq;
    win.na = x.n_sink;
    win.b0 = a.w_sink + x.vq;
    win.nb = x.win - x.n_sink;
    const int quota = (int)((uint32_t)(x.tiles + n_chunks * x.cost + n_splits - 1) / (uint32_t)n_splits);
    win_tiles = quota > x.cost ? quota - x.cost : 0;
    const int most = n_chunks > 0 ? (int)((uint32_t)x.tiles / (uint32_t)n_chunks) : win_tiles;
    win_tiles = win_tiles > most ? most : win_tiles;
    const int rest = x.tiles - n_chunks * win_tiles, others = n_splits - n_chunks;
    base_t = (int)((uint32_t)rest / (uint32_t)others);
    rem_t = rest - base_t * others;
  }
  const long long bh = (long long)b * a.n_kv_heads + hk;
  constexpr bool has_kz = ZK, has_vz = ZV != 0;  // zero-point arrays exist unless the tensor is symmetric-only
  constexpr bool late_vz = ZV == 2;              // value zero-points: only where flagged, at the start of their tile

  // ---- tile range of this wavefront.  The first win.n_chunks wavefronts of a (batch, kv-head)
  // also serve one chunk of the fp16 windows each (after their tiles) and get win_tiles tiles;
  // the others share the remaining tiles evenly.
  const int n_tiles = (n_both + TILE - 1) / TILE;
  const int s_idx = ALONE ? group : wave * n_groups + group;   // (the chunks go to different work-groups first)
  int t0 = 0, t1 = 0;
  if (!ALONE && s_idx >= n_splits) {                     // (a launch that leaves its partials to the merge: beyond the plan)
  } else if (s_idx < win.n_chunks) {
    t0 = s_idx * win_tiles;
    t1 = t0 + win_tiles;
  } else {
    const int j = s_idx - win.n_chunks;                  // base_t, rem_t: (n_tiles - n_chunks * win_tiles) divided by the plain wavefronts
    t0 = win.n_chunks * win_tiles + j * base_t + (j < rem_t ? j : rem_t);
    t1 = t0 + base_t + (j < rem_t ? 1 : 0);
  }

  // Operand tables, a head's row padded by 16 bytes (four heads' rows then start in different banks).  The query's, the
  // group sums and the zeros stand once for the work-group; a wavefront's own part holds its probability tables, then the
  // window pass's memory, then its state for the join.
  using L = Lds<KB, VB, G, NH4>;
  constexpr int QS = L::QS, PS = L::PS, ZEROS = L::ZEROS;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  _Float16* tables = reinterpret_cast<_Float16*>(lds);
  constexpr int QA = 0;                       // query operand table [head][word][mfma][slot]
  constexpr int QA1 = QA + NH * QS;           // the same for the plane of high bits (1-bit fields, weight 4)
  constexpr int ZERO = QA1 + (HIK ? NH * QS : 0);        // zeros, for any table
  float* coef_lds = reinterpret_cast<float*>(lds + L::COEF);                     // [NH]
  float (*qsum)[NG][4] = reinterpret_cast<float (*)[NG][4]>(lds + L::QSUM);      // [NH4] log2e/sqrt(d) * sum of q over each key group
  const int own_lds = L::SHARED + wave * L::OWN;         // bytes
  const int PA = own_lds / 2;                 // probability operand table [head][word][mfma][slot]
  const int PA1 = PA + NH * PS;               // ... and its high bits' one

  WaveState<NH> part;
#pragma unroll
  for (int h = 0; h < NH; ++h) { part.m[h] = -INFINITY; part.l[h] = 0.f; part.o[h] = float2{0.f, 0.f}; }   // (an empty partial)
  // ---- per-(b, hk) base pointers
  const long long slab = kPagedStore ? 0 : bh * a.capacity;             // first store row of (b, hk); paged: see below
  const uint8_t* kcodes_slab = a.k.codes + slab * (D * KB / 8);
  const __half* kscales_slab = a.k.scales + slab * NG;
  const __half* kzeros_slab = has_kz ? a.k.zeros + slab * NG : nullptr;
  const long long vgroups = slab / G;
  const uint8_t* vcodes_slab = a.v.codes + vgroups * D * (G * VB / 8);
  const __half* vscales_slab = a.v.scales + vgroups * D;
  const __half* vzeros_slab = has_vz ? a.v.zeros + vgroups * D : nullptr;
  const int last_row = n_both - 1, last_group = n_both / G - 1;
  constexpr int ROWB = D * KB / 8;                     // bytes of one key row
  constexpr int GB = G * VB / 8;                       // bytes of one channel of one value group

  // Paged store: a tile is one page (kPageTokens == TILE), so the tile's rows sit `shift` rows away
  // from where the contiguous layout of a pool-sized cache would put rows tile * 64 .. of (b = 0, hk = 0):
  // a wave-uniform 64-bit shift of the six bases, looked up once per tile.
  static_assert(kPageTokens == TILE, "a page of the store is one tile of this kernel");
  // The table entries of this wavefront's tiles come in one vector load, lane i holding the entry of
  // tile pages_from + i (a wavefront with more than 64 tiles reloads every 64), and a tile reads its
  // entry with a lane read.  (A scalar load per tile, even issued a tile ahead, costs more: scalar loads
  // return out of order, so the first wait for an LDS operation behind it waits for the load as well.)
  constexpr bool paged = kPagedStore;
  int pages_from = t0, pages_held = 0;
  auto fetch_pages = [&](int from) {
    const int tile = from + lane < t1 ? from + lane : t1 - 1;
    pages_from = from;
    pages_held = a.pages.table[(long long)b * a.pages.tiles_per_seq + tile];
  };
  if constexpr (paged) {
    if (t1 > t0) fetch_pages(t0);
  }

  // All offsets inside one (b, hk) slab fit 32 bits; bases are wave-uniform.
  auto load_tile = [&](int tile, Regs& t) {
    const uint8_t *kcodes = kcodes_slab, *vcodes = vcodes_slab;
    const __half *kscales = kscales_slab, *kzeros = kzeros_slab, *vscales = vscales_slab, *vzeros = vzeros_slab;
    if constexpr (paged) {
      if (tile - pages_from >= 64) fetch_pages(tile);
      int page = __builtin_amdgcn_readlane(pages_held, tile - pages_from);
      page = page < 0 ? 0 : (page >= a.pages.pool_pages ? a.pages.pool_pages - 1 : page);
      const long long shift = (((long long)page * a.n_kv_heads + hk) - tile) * TILE, gshift = shift / G * D;
      kcodes += shift * ROWB; kscales += shift * NG;
      if constexpr (has_kz) kzeros += shift * NG;
      vcodes += gshift * GB; vscales += gshift;
      if constexpr (has_vz) vzeros += gshift;
      t.gshift = gshift;
    }
    int row = tile * TILE + lane;
    row = row > last_row ? last_row : row;
    const u32x4* kp = reinterpret_cast<const u32x4*>(kcodes + (uint32_t)row * ROWB);
#pragma unroll
    for (int i = 0; i < KC; ++i) t.kc[i] = stream_load(kp + i);
    if constexpr (NG == 4) {
      const u32x2 s = stream_load(reinterpret_cast<const u32x2*>(kscales + (uint32_t)row * NG));
      t.ks[0] = s.x; t.ks[1] = s.y;
      if constexpr (has_kz) {
        const u32x2 z = stream_load(reinterpret_cast<const u32x2*>(kzeros + (uint32_t)row * NG));
        t.kz[0] = z.x; t.kz[1] = z.y;
      }
    } else {
      t.ks[0] = stream_load(reinterpret_cast<const uint32_t*>(kscales + (uint32_t)row * NG));
      if constexpr (has_kz) t.kz[0] = stream_load(reinterpret_cast<const uint32_t*>(kzeros + (uint32_t)row * NG));
    }
#pragma unroll
    for (int gi = 0; gi < GPT; ++gi) {
      int grp = tile * GPT + gi;
      grp = grp > last_group ? last_group : grp;
      const uint32_t ch = (uint32_t)grp * D + 2 * lane;
      if constexpr (VW % 4 == 0) {
        const u32x4* vp = reinterpret_cast<const u32x4*>(vcodes + ch * GB);
#pragma unroll
        for (int i = 0; i < VW / 4; ++i) {
          const u32x4 v = stream_load(vp + i);
          t.vw[gi][4 * i] = v.x; t.vw[gi][4 * i + 1] = v.y; t.vw[gi][4 * i + 2] = v.z; t.vw[gi][4 * i + 3] = v.w;
        }
      } else {                                          // 3-bit, G = 32: 24 bytes per lane
        const u32x2* vp = reinterpret_cast<const u32x2*>(vcodes + ch * GB);
#pragma unroll
        for (int i = 0; i < VW / 2; ++i) {
          const u32x2 v = stream_load(vp + i);
          t.vw[gi][2 * i] = v.x; t.vw[gi][2 * i + 1] = v.y;
        }
      }
      t.vs[gi] = stream_load(reinterpret_cast<const uint32_t*>(vscales + ch));
      if constexpr (has_vz && !late_vz) t.vz[gi] = stream_load(reinterpret_cast<const uint32_t*>(vzeros + ch));
    }
  };

  // ---- the query loads go out first (the set-up below waits for them), the first tile's loads
  // right behind them: those overlap the query set-up.  One wavefront sets four heads up for the whole work-group (the last
  // ones, which carry no window chunk); the others meet it at the barrier with their first tile in flight.
  struct Query {
    u32x4 raw[NH4];
    float4_t fac[NH4][2];                              // per-channel query factors, when given
  };
  auto sets_up = [&](int rnd) { return ALONE || wave == waves - 1 - (waves > rnd ? rnd : 0); };
  auto load_query = [&](Query& q) {
#pragma unroll
  for (int rnd = 0; rnd < NH4; ++rnd) {
    if (!sets_up(rnd)) continue;
    const int h = (rnd * 64 + lane) / (D / 8), c0 = 8 * ((rnd * 64 + lane) % (D / 8));
    q.raw[rnd] = u32x4{0u, 0u, 0u, 0u};
    if (h < r) q.raw[rnd] = *reinterpret_cast<const u32x4*>(a.q + ((long long)b * a.n_q_heads + hk * r + h) * D + c0);
    if (a.q_scale) {
      q.fac[rnd][0] = *reinterpret_cast<const float4_t*>(a.q_scale + hk * D + c0);
      q.fac[rnd][1] = *reinterpret_cast<const float4_t*>(a.q_scale + hk * D + c0 + 4);
    }
  }
  };

  // ---- query: fp16 (optionally rescaled), offset factors folded in.  A lane takes 8
  // consecutive channels of one head (one 16-byte load); the channels of one key group sit in
  // G/8 neighbouring lanes, so the group sums of q come from a few DPP adds.
  float q_coef[4];                                       // the score's constants of this lane's four heads
  auto set_up = [&](const Query& q) {
#pragma unroll
  for (int rnd = 0; rnd < NH4; ++rnd) {
    if (!sets_up(rnd)) continue;
    const int idx = rnd * 64 + lane;
    const int h = idx / (D / 8), c0 = 8 * (idx % (D / 8));
    const uint32_t rw[4] = {q.raw[rnd].x, q.raw[rnd].y, q.raw[rnd].z, q.raw[rnd].w};
    float qv[8], part = 0.f, mx = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t hb = (e & 1) ? (rw[e / 2] >> 16) : (rw[e / 2] & 0xffffu);
      qv[e] = __half2float(__ushort_as_half((unsigned short)hb));
      if (a.q_scale) qv[e] = __half2float(scaled_half(qv[e], q.fac[rnd][e / 4][e % 4]));
      part += qv[e];
      mx = __builtin_fmaxf(mx, __builtin_fabsf(qv[e]));
    }
    // power of two that brings the head's largest |q| into [2^8, 2^9): with factors of 2^-2 and more the
    // table entries stay normal fp16 numbers down to 2^-20 of the head's maximum whatever the magnitude of the
    // queries (a head is D/8 = 16 neighbouring lanes)
    static_assert(D / 8 == 16, "a head is one 16-lane row of the cross-lane operations below");
    mx = __builtin_fmaxf(mx, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, mx), 0xB1, 0xF, 0xF, true)));    // lane ^ 1
    mx = __builtin_fmaxf(mx, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, mx), 0x4E, 0xF, 0xF, true)));    // lane ^ 2
    mx = __builtin_fmaxf(mx, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, mx), 0x141, 0xF, 0xF, true)));   // mirror within 8
    mx = __builtin_fmaxf(mx, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, mx), 0x140, 0xF, 0xF, true)));   // mirror within 16
    const int q_exp = mx > 0.f ? (int)((__float_as_uint(mx) >> 23) & 0xffu) - 127 : 8;
    const float q_pow = __uint_as_float((uint32_t)(127 + 8 - q_exp) << 23);
    // per-head constant of the score, log2e/sqrt(d) * 2^(24 - CK) / (the head's factor)
    const float coef = (kSmScale * kLog2e * (float)(1 << (24 - CK))) * __uint_as_float((uint32_t)(127 - 8 + q_exp) << 23);
    if constexpr (ALONE) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float of_head = from_lane(coef, 16 * j);
        q_coef[j] = rnd == 0 || (lane & 16) ? of_head : q_coef[j];
      }
    } else if (lane % 16 == 0) {
      coef_lds[h] = coef;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = c0 + e;
      const int word = c / FK::FPW, ep = c % FK::FPW;
      const int f = ep % FK::HALF;
      const float factor = (float)(1 << CK) / (float)(1 << FK::off(f));
      tables[QA + h * QS + word * (MPWK * 4) + FK::slot(ep)] = (_Float16)(qv[e] * q_pow * factor);
      if constexpr (HIK) {
        const int word1 = c / 32, ep1 = c % 32;
        const float factor1 = (float)(4 << CK) / (float)(1 << F1::off(ep1 % 16 % F1PER));
        tables[QA1 + h * QS + word1 * (F1::MPW * 4) + F1::slot(ep1)] = (_Float16)(qv[e] * q_pow * factor1);
      }
    }
    // sum over the G/8 lanes of the group (4 lanes: one quad; 8 lanes: two quads)
    part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0xB1, 0xF, 0xF, true));
    part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0x4E, 0xF, 0xF, true));
    if constexpr (G == 64)
      part += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, part), 0x141, 0xF, 0xF, true));
    if ((idx % (G / 8)) == 0) qsum[h / 4][c0 / G][h % 4] = part * (kSmScale * kLog2e);
  }
  };
  auto meet = [] {
    if constexpr (ALONE) wave_fence();
    else __syncthreads();
  };
  int* arrivals = reinterpret_cast<int*>(lds + L::COUNT);
  auto clear = [&] {
    if (JOIN && lane == 0) *arrivals = 0;
    for (int i = 2 * lane; i < ZEROS; i += 128) *reinterpret_cast<uint32_t*>(&tables[ZERO + i]) = 0u;
  };
  if (!ALONE && wave == 0) clear();
  // A wavefront without a tile (a launch with more wavefronts than tiles gives the window chunks wavefronts of their own)
  // meets the others behind the loads of its window chunk.
  const bool has_tiles = t1 > t0, has_chunk = s_idx < win.n_chunks;
  Query query;
  if (!has_tiles) {
    if constexpr (!ALONE) {                              // (alone, it needs no tables)
      if (waves > 1) {
        load_query(query);
        set_up(query);
      }
      if (!has_chunk) __syncthreads();
    }
  } else {
  // (the first tile's loads and their use in one branch: brought together from two, they were waited for at the barrier,
  // 0.9 us of a launch of 1024 wavefronts with a few tiles each)
  Regs bufA, bufB;
  load_query(query);
  load_tile(t0, bufA);
  set_up(query);
  if constexpr (ALONE) clear();
  meet();
  // Four results a lane: heads 4 par .. 4 par + 3 (see CH below); their constants of the score.
  const int par = NH4 == 2 ? (lane >> 4) & 1 : 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (ALONE) continue;
    q_coef[i] = coef_lds[4 * par + i];
    if constexpr (NH4 == 1) q_coef[i] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, q_coef[i])));
  }

  // ---- A operands of the zero-point term: sum over groups of Zeff_g * (sum of q over group g) is a
  // 4 (heads) x 4 (groups) product per token, one more matrix instruction.  The group sums of q
  // enter as two fp16 pieces (hi + lo, 2^-22 relative) so that the term keeps fp32 accuracy; Zeff
  // is an exact fp16 number (Z for an asymmetric group, -2^(b-1) S for a symmetric one).  The
  // operands carry 2 * qsum and Zeff / 2: S is at most 65504 / (2^(b-1) - 1), so 2^(b-2) S is
  // finite in fp16 for every finite cache where 2^(b-1) S is not; Z / 2 is exact unless Z is an fp16
  // denormal with an odd last bit (2^-25 off).
  half4_t qs_hi, qs_lo;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float v = g < NG ? 2.f * qsum[par][g][lane & 3] : 0.f;
    const _Float16 hi = (_Float16)v;
    qs_hi[g] = hi;
    qs_lo[g] = (_Float16)(v - (float)hi);
  }

  // ---- running softmax state (log2 domain) and output accumulators.
  // m_run is a reference level, not the exact running maximum: it is raised (and l, o rescaled)
  // only when some score exceeds it by more than kSlack, so the common tile pays no wave-wide
  // reduction and no rescale.  Probabilities are then at most 2^kSlack, times a factor of at most
  // 2^(CV - 2): still inside fp16.  l_run and o are kept in the raw scale of the matrix results.
  // The first tile sets the level to its exact maximum.
  constexpr float kSlack = HIV ? 5.0f : 6.0f;           // (the high-bit plane's factors reach 2^CV)
  float m_run[4], l_run[4], o[CH][2][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m_run[i] = 0.f;
    l_run[i] = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) o[c][0][i] = o[c][1][i] = 0.f;
  }

  // Column (token, or channel pair) of chain c in this lane.
  auto column = [&](int c) { return CH == 1 ? lane : (lane & ~16) + 16 * c; };
  // where the lane's tokens sit in the probability operand table, and their offset factor (the same for both chains)
  const int p_e = column(0) % FV::FPW;
  const float p_shift = (float)(CV - FV::off(p_e % FV::HALF));              // p is stored as p * 2^(CV - off)
  auto p_index = [&](int c) { const int t = column(0); return t / FV::FPW * (MPWV * 4) + FV::slot(t % FV::FPW) + 16 * c; };
  // the same in the high-bit plane's table: p * 4 * 2^(CV - off), as a factor on the stored p
  const int p1_e = column(0) % 32;
  const float p1_factor = __builtin_amdgcn_exp2f((float)(CV + 2 - F1::off(p1_e % 16 % F1PER)) - p_shift);
  auto p1_index = [&](int c) { const int t = column(0); return t / 32 * (F1::MPW * 4) + F1::slot(t % 32) + c; };   // (16 tokens on: the other half of the word)
  // A operand of the 16x16x32 instructions: row l % 16, entries 8 (l / 16) .. + 7 of the contraction.
  // Four heads: the matrix is block diagonal -- rows 4 j .. 4 j + 3 are the four heads, with entries only where block j of
  // the contraction is -- so that lane l's result is its own column's product with its own eight B entries for the four
  // heads (block j = l / 16 of rows 4 j ..).
  // Eight heads: two blocks, rows 8 j .. 8 j + 7 the eight heads, 16 contraction indices each: a column's B entries stand in
  // the lanes l and l + 16 (the first half of a group's indices in the first), a chain of instructions takes 32 columns,
  // and lane l's result are heads 4 par .. 4 par + 3 of its chain's column.  Half the matrix instructions of eight
  // heads as twice four, and a quarter of the operand reads; the halves of two columns change places by one lane swap a word.
  // (Eight query heads per kv head, step before -> now: 8 x 8 x 32k tokens, 2-bit 51.8 us -> 45.5, 4-bit 86.3 -> 77.1; 32 x 8 x
  // 8k, G = 64 51.6 -> 39.9; attention call, 4 x 8 x 16k, 3-bit keys 27.5 -> 23.6.)
  // Lanes off the diagonal read the zeros.
  const bool diagonal = CH == 1 ? ((lane >> 2) & 3) == (lane >> 4) : ((lane >> 3) & 1) == (lane >> 5);
  const int head_row = lane & (NH - 1), half_at = CH == 1 ? 0 : par * (G / 2);
  const int qa = diagonal ? QA + head_row * QS + half_at : ZERO, pa = diagonal ? PA + head_row * PS + half_at : ZERO;
  const int qa1 = diagonal ? QA1 + head_row * QS + half_at : ZERO, pa1 = diagonal ? PA1 + head_row * PS + half_at : ZERO;
  // the same instruction with all blocks alike (row r = head r % NH) sums 32 table entries for every lane at once
  const int pl_lane = PA + head_row * PS + 8 * (lane >> 4);
  const half8_t ones = ones_operand<LBV>(lane >> 4);
  auto a_operand = [&](int base, int entry) -> half8_t { return *reinterpret_cast<const half8_t*>(&tables[base + entry]); };

  // A word of each chain's column: of this lane's column (four heads); from words `lo` and `hi` of the lane's own column,
  // the half that this lane takes of both chains' columns (eight heads).
  struct Chains { uint32_t w[CH]; };
  auto chains = [&](uint32_t lo, uint32_t hi) -> Chains {
    if constexpr (CH == 1) {
      return Chains{{lo}};
    } else {
      const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(lo, hi, false, false));
      return Chains{{r.x, r.y}};
    }
  };
  // ... the same word of both chains' columns
  auto both = [&](uint32_t w) -> Chains {
    uint32_t copy = w;
    if constexpr (CH == 2) asm volatile("" : "+v"(copy));   // (a register of its own)
    return chains(w, copy);
  };

  // The query operands stay in registers where they fit (64 for four heads, 32 for 2-bit keys and eight): read from the
  // table tile by tile, each matrix instruction of the score pass waits for its own LDS read.
  constexpr bool QREG = CH == 1 || KB == 2;
  constexpr int KOPS = D / 8 / CH;                       // matrix instructions per chain and (low) plane of a key row
  half8_t q_op[QREG ? KOPS : 1];
  if constexpr (QREG) {
#pragma unroll
    for (int i = 0; i < KOPS; ++i) {
      u32x4 v = __builtin_bit_cast(u32x4, a_operand(qa, CH == 1 ? 8 * i : 8 * i / (G / 2) * G + 8 * i % (G / 2)));
      asm volatile("" : "+v"(v));                        // (not to be read again)
      q_op[i] = __builtin_bit_cast(half8_t, v);
    }
  }

  auto process = [&](const Regs& cur, int tile, bool first) {
    // sparse value zero-points: the lanes whose scale pair carries a flag fetch theirs now; they are
    // needed at the end of the tile
    uint32_t vz_late[GPT];
    if constexpr (late_vz) {
      const __half* vz_tile = vzeros_slab;
      if constexpr (paged) vz_tile += cur.gshift;
#pragma unroll
      for (int gi = 0; gi < GPT; ++gi) {
        int grp = tile * GPT + gi;
        grp = grp > last_group ? last_group : grp;
        vz_late[gi] = 0u;
        if (cur.vs[gi] & 0x80008000u)
          vz_late[gi] = stream_load(reinterpret_cast<const uint32_t*>(vz_tile + (uint32_t)grp * D + 2 * lane));
      }
    }
    // ================= scores: lane = token (Eq. att:1 with Eq. hybrid_dequant fused) =================
    // one MFMA chain per key group (and columns), the chains interleaved so that consecutive MFMAs are independent
    float4_t acc[NG][CH];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < CH; ++c) acc[g][c] = float4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int HWK = WPGK / CH;                       // words of a group that a lane takes
#pragma unroll
    for (int wd = 0; wd < HWK; ++wd) {
      Shifted<LBK> w[NG][CH];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const Chains x = chains(cur.k_word(g * WPGK + wd), cur.k_word(g * WPGK + (CH - 1) * HWK + wd));
#pragma unroll
        for (int c = 0; c < CH; ++c) w[g][c] = Shifted<LBK>(x.w[c]);
      }
#pragma unroll
      for (int m = 0; m < MPWK; m += 2) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
          for (int c = 0; c < CH; ++c)
            acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                QREG ? q_op[QREG ? (g * (G / CH) + wd * FK::FPW + 4 * m) / 8 : 0] : a_operand(qa, g * G + wd * FK::FPW + 4 * m),
                operand<LBK>(w[g][c], m), acc[g][c], 0, 0, 0);
      }
    }
    if constexpr (HIK) {
      // the plane of high bits joins the same chains: its query table carries the weight 4
      constexpr int HW1 = HWG / CH > 0 ? HWG / CH : 1, M1 = HWG >= CH ? F1::MPW : F1::MPW / 2;
#pragma unroll
      for (int j = 0; j < HW1; ++j) {
        Shifted<1> w[NG][CH];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const Chains x = HWG >= CH ? chains(cur.k_high(g * HWG + j), cur.k_high(g * HWG + (CH - 1) * HW1 + j)) : both(cur.k_high(g * HWG + j));
#pragma unroll
          for (int c = 0; c < CH; ++c) w[g][c] = Shifted<1>(HWG >= CH ? x.w[c] : x.w[c] >> (8 * par));
        }
#pragma unroll
        for (int m = 0; m < M1; m += 2) {
#pragma unroll
          for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int c = 0; c < CH; ++c)
              acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  a_operand(qa1, (g * HWG + j) * 32 + 4 * m), operand<1>(w[g][c], m), acc[g][c], 0, 0, 0);
        }
      }
    }
    // e[c][i] = score (log2 domain) + offset shift - reference level: the exponent of the stored probability.
    // Per group: |S| * (raw inner sum) + Zeff * (sum of q).  The scale sign bit marks an asymmetric
    // group, so max(s, 0) is |S| for a symmetric group and 0 for an asymmetric one, and
    // Zeff = Z - 2^(b-1) * max(s, 0) needs no select (Z is stored as +0 for symmetric groups).
    // Scales and zero-points enter the FMAs as fp16 sources; the constant factor is applied once.
    float e[CH][4];
    uint32_t ks[NG / 2][CH];
#pragma unroll
    for (int gp = 0; gp < NG / 2; ++gp) {
      const Chains x = both(cur.ks[gp]);
#pragma unroll
      for (int c = 0; c < CH; ++c) ks[gp][c] = x.w[c];
    }
    {
      // Zeff / 2 of the lane's own token's groups as fp16: Z / 2 - 2^(b-2) max(s, 0) (one of the two terms is 0)
      u32x2 zw[CH];
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) {
        Chains x = {};
        if (gp < NG / 2) {
          const half2_t sp = __builtin_bit_cast(half2_t, cur.ks[gp < NG / 2 ? gp : 0]);
          half2_t zp;
          constexpr _Float16 kNegQuarterK = (_Float16)(-HALFK / 2), kHalf = (_Float16)0.5f;
          if constexpr (has_kz)
            zp = positive_part(sp) * half2_t{kNegQuarterK, kNegQuarterK} + __builtin_bit_cast(half2_t, cur.kz[gp < NG / 2 ? gp : 0]) * half2_t{kHalf, kHalf};
          else zp = sp * half2_t{kNegQuarterK, kNegQuarterK};
          x = both(__builtin_bit_cast(uint32_t, zp));
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) zw[c][gp] = x.w[c];
      }
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const half4_t zop = __builtin_bit_cast(half4_t, zw[c]);
        float4_t ez = float4_t{p_shift - m_run[0], p_shift - m_run[1], p_shift - m_run[2], p_shift - m_run[3]};
        ez = __builtin_amdgcn_mfma_f32_4x4x4f16(qs_hi, zop, ez, 0, 0, 0);
        ez = __builtin_amdgcn_mfma_f32_4x4x4f16(qs_lo, zop, ez, 0, 0, 0);
        e[c][0] = ez.x; e[c][1] = ez.y; e[c][2] = ez.z; e[c][3] = ez.w;
      }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const float S = __builtin_fabsf((float)half_of(ks[g / 2][c], g & 1));
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = __builtin_fmaf(S, acc[g][c][i], t[i]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) e[c][i] = __builtin_fmaf(q_coef[i], t[i], e[c][i]);   // undoes the operand factors and the head's query factor
    }

    // ================= running softmax (Eq. att:2), probabilities to the operand table =================
    if (tile * TILE + (TILE - 1) > last_row) {         // ragged last tile: columns past the end weigh nothing
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const bool valid = tile * TILE + column(c) <= last_row;
#pragma unroll
        for (int i = 0; i < 4; ++i) e[c][i] = valid ? e[c][i] : -INFINITY;
      }
    }
    bool raise = false;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) raise |= e[c][i] > kSlack + p_shift;
    if (first || __builtin_amdgcn_ballot_w64(raise) != 0) {   // rare after the first tiles
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // largest score relative to the current level
        const float mx = CH == 1 ? wave_max(e[0][i] - p_shift) : parity_max(fmaxf(e[0][i], e[CH - 1][i]) - p_shift, par);
        const float d = first ? mx : fmaxf(mx, 0.f);         // the level only rises, except when it is first set
        const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-d);
        m_run[i] += d;
        l_run[i] *= alpha;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          e[c][i] -= d;
          o[c][0][i] *= alpha;
          o[c][1][i] *= alpha;
        }
      }
    }
    wave_fence();                                      // previous tile's readers of pA are done
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(e[c][i]);
        tables[PA + (4 * par + i) * PS + p_index(c)] = (_Float16)p;
        if constexpr (HIV) tables[PA1 + (4 * par + i) * PS + p1_index(c)] = (_Float16)(p * p1_factor);
      }
    wave_fence();

    // ================= values: lane = two channels (Eq. att:3 with Eq. hybrid_dequant fused) =================
#pragma unroll
    for (int gi = 0; gi < GPT; ++gi) {
      float4_t av[CH][2], accl = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < CH; ++c) av[c][0] = av[c][1] = float4_t{0.f, 0.f, 0.f, 0.f};
      constexpr int HWV = WPGV / CH;
#pragma unroll
      for (int wd = 0; wd < HWV; ++wd) {
        Shifted<LBV> w[2][CH];
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
          const Chains x = chains(cur.v_word(gi, ch, wd), cur.v_word(gi, ch, (CH - 1) * HWV + wd));
#pragma unroll
          for (int c = 0; c < CH; ++c) w[ch][c] = Shifted<LBV>(x.w[c]);
        }
#pragma unroll
        for (int m = 0; m < MPWV; m += 2) {
          const half8_t aop = a_operand(pa, gi * G + wd * FV::FPW + 4 * m);
#pragma unroll
          for (int ch = 0; ch < 2; ++ch)
#pragma unroll
            for (int c = 0; c < CH; ++c)
              av[c][ch] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aop, operand<LBV>(w[ch][c], m), av[c][ch], 0, 0, 0);
        }
      }
#pragma unroll
      for (int x = 0; x < G; x += 32)
        accl = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_operand(pl_lane, gi * G + x), ones, accl, 0, 0, 0);
      if constexpr (HIV) {
        constexpr int HW1 = HWG / CH > 0 ? HWG / CH : 1, M1 = HWG >= CH ? F1::MPW : F1::MPW / 2;
#pragma unroll
        for (int j = 0; j < HW1; ++j) {
          Shifted<1> w[2][CH];
#pragma unroll
          for (int ch = 0; ch < 2; ++ch) {
            const Chains x = HWG >= CH ? chains(cur.v_high(gi, ch, j), cur.v_high(gi, ch, (CH - 1) * HW1 + j)) : both(cur.v_high(gi, ch, j));
#pragma unroll
            for (int c = 0; c < CH; ++c) w[ch][c] = Shifted<1>(HWG >= CH ? x.w[c] : x.w[c] >> (8 * par));
          }
#pragma unroll
          for (int m = 0; m < M1; m += 2) {
            const half8_t aop = a_operand(pa1, (gi * HWG + j) * 32 + 4 * m);
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
              for (int c = 0; c < CH; ++c)
                av[c][ch] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aop, operand<1>(w[ch][c], m), av[c][ch], 0, 0, 0);
          }
        }
      }
      // accl = 2^(CV - 24) * (sum of the fp16 probabilities of this group); l and o stay in that scale
#pragma unroll
      for (int i = 0; i < 4; ++i) l_run[i] += accl[i];
      const Chains sx = both(cur.vs[gi]);
      Chains zx = {};
      if constexpr (has_vz) zx = both(late_vz ? vz_late[gi] : cur.vz[gi]);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t spair = sx.w[c];
        const float S0 = __builtin_fabsf((float)half_of(spair, 0)), S1 = __builtin_fabsf((float)half_of(spair, 1));
        float z0, z1;
        if constexpr (has_vz) {
          const uint32_t mpair = __builtin_bit_cast(uint32_t, positive_part(__builtin_bit_cast(half2_t, spair)));
          z0 = __builtin_fmaf((float)half_of(mpair, 0), (float)(-HALFV), (float)half_of(zx.w[c], 0));
          z1 = __builtin_fmaf((float)half_of(mpair, 1), (float)(-HALFV), (float)half_of(zx.w[c], 1));
        } else {
          z0 = S0 * (float)(-HALFV);
          z1 = S1 * (float)(-HALFV);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          o[c][0][i] = __builtin_fmaf(S0, av[c][0][i], __builtin_fmaf(z0, accl[i], o[c][0][i]));
          o[c][1][i] = __builtin_fmaf(S1, av[c][1][i], __builtin_fmaf(z1, accl[i], o[c][1][i]));
        }
      }
    }
  };

  // ---- two register buffers, ping-pong: the next tile's loads are in flight while this one is computed
  {
    const int n = t1 - t0;
    int i = 0;
    // (one or two tiles only: ahead of the wavefronts that carry nothing but a window chunk)
    if (n <= 2) __builtin_amdgcn_s_setprio(2);
    while (i + 2 < n) {
      // the wavefront that is behind gets the SIMD first: the two wavefronts of a SIMD then
      // finish together instead of one running alone (and at a lower rate) at the end
      if (4 * i < n) __builtin_amdgcn_s_setprio(3);
      else if (2 * i < n) __builtin_amdgcn_s_setprio(2);
      else if (4 * i < 3 * n) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
      load_tile(t0 + i + 1, bufB);
      process(bufA, t0 + i, i == 0);
      load_tile(t0 + i + 2, bufA);
      process(bufB, t0 + i + 1, false);
      i += 2;
    }
    if (n - i == 2) {
      load_tile(t0 + i + 1, bufB);
      process(bufA, t0 + i, i == 0);
      process(bufB, t0 + i + 1, false);
    } else if (n - i == 1) {
      process(bufA, t0 + i, i == 0);
    }
  }

  // ---- this wavefront's state over its tiles: every head of the lane's own channels
  constexpr float kUndo = (float)(1 << (24 - CV));     // the operand factors of the value pass
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (CH == 1) {
      part.o[i].x = o[0][0][i] * kUndo;
      part.o[i].y = o[0][1][i] * kUndo;
      part.m[i] = m_run[i];
      part.l[i] = l_run[i] * kUndo;
    } else {
      const Chains x = chains(__float_as_uint(o[0][0][i] * kUndo), __float_as_uint(o[CH - 1][0][i] * kUndo));
      const Chains y = chains(__float_as_uint(o[0][1][i] * kUndo), __float_as_uint(o[CH - 1][1][i] * kUndo));
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        part.o[4 * c + i] = float2{__uint_as_float(x.w[c]), __uint_as_float(y.w[c])};
        part.m[4 * c + i] = from_lane(m_run[i], 16 * c);
        part.l[4 * c + i] = from_lane(l_run[i] * kUndo, 16 * c);
      }
    }
  }
  }

  // ---- the window chunk of this wavefront joins it
  if (has_chunk) {
    __builtin_amdgcn_s_setprio(0);
    WaveState<NH> w;
    window_pass<NH4, KB, G, true, false, kPagedStore>(a, bh, win.na, win.b0, win.nb, s_idx, win.n_chunks, 0, lds + own_lds, w,
                                                      [&] { if (!ALONE && !has_tiles) __syncthreads(); });
    if (!JOIN) store_partial(a, w, bh, r, n_splits + s_idx, lane);
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      if (!JOIN) continue;
      const float top = fmaxf(part.m[h], w.m[h]);
      const float f = level_weight(part.m[h], top), g = level_weight(w.m[h], top);
      part.m[h] = top;
      part.l[h] = part.l[h] * f + w.l[h] * g;
      part.o[h].x = part.o[h].x * f + w.o[h].x * g;
      part.o[h].y = part.o[h].y * f + w.o[h].y * g;
    }
  }

  // ---- the append of the step's token: disjoint memory.  The wavefront of one work-group that is through first takes it,
  // while the others still have tiles.
#if INNERQ_INNER_JOIN
  if (appends && group == n_groups - 1) {
    int at = 0;
    if (lane == 0) at = __hip_atomic_fetch_add(arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_readfirstlane(at) == 0) append_keys_and_copies<G, KB>(append, bh, a.n_tokens - 1, lane);
  }
#endif

  if constexpr (!JOIN) {                                 // partials for a later launch (the tiles' after the chunk's: nothing reuses its registers)
    if (s_idx < n_splits) store_partial(a, part, bh, r, s_idx, lane);
  } else {
    // ---- the work-group's wavefronts, and the sequence-head's work-groups, meet
    join_and_store<NH>(a, part, reinterpret_cast<float*>(lds + L::SHARED), L::OWN / 4, wave, waves, lane, bh, r, group, n_groups);
  }
}

template <int KB, int VB, int G, bool ZK, int ZV>
hipError_t launch_z(const AttnArgs& a, int n_both, int n_splits, const WindowSet& win, const Launch& L) {
  const int r = a.n_q_heads / a.n_kv_heads;
  // A window chunk costs its wavefront about as much time as window_cost() tiles: the wavefronts
  // that carry one get that many tiles fewer than the common quota.
  const int n_tiles = (n_both + TILE - 1) / TILE;
  const int cost = win.n_chunks > 0 ? window_cost((win.na + win.nb + win.n_chunks - 1) / win.n_chunks, G) : 0;
  const int quota = (n_tiles + win.n_chunks * cost + n_splits - 1) / n_splits;
  int win_tiles = quota > cost ? quota - cost : 0;
  if (win.n_chunks > 0 && win_tiles > n_tiles / win.n_chunks) win_tiles = n_tiles / win.n_chunks;
  if (L.waves < 1 || L.waves > kJoinWaves || (a.join && n_splits > kJoinGroups * L.waves) || (!a.join && L.append)) return hipErrorInvalidValue;
  if (!JOIN && L.waves > 1 && (r <= 4 || a.n_dev)) return hipErrorInvalidValue;   // (not built)
  if (n_splits <= win.n_chunks) return hipErrorInvalidValue;      // the host gives at least one plain wavefront
  if (a.batch > 65535 || a.n_kv_heads > 65535) return hipErrorInvalidValue;
  const int rest = n_tiles - win.n_chunks * win_tiles, others = n_splits - win.n_chunks;
  const int base_t = rest / others, rem_t = rest % others;
  dim3 grid((unsigned)((n_splits + L.waves - 1) / L.waves), (unsigned)a.n_kv_heads, (unsigned)a.batch);
  if (a.shared_groups > 0) grid = dim3((unsigned)a.shared_groups, (unsigned)a.n_kv_heads, 1u);
  const unsigned lds_bytes = (unsigned)(r <= 4 ? Lds<KB, VB, G, 1>::bytes(L.waves) : Lds<KB, VB, G, 2>::bytes(L.waves));
  // (the launch with dispatch events only when events were asked for: the plain launch is the one a
  // stream capture is sure to record)
  const bool timed = L.ev_start || L.ev_stop;
  const int appends = L.append ? 1 : 0;
  auto go = [&](auto kernel, auto q) {
    if (timed)
      hipExtLaunchKernelGGL(kernel, grid, dim3(64u * L.waves), lds_bytes, L.stream, L.ev_start, L.ev_stop, 0, a, n_both, n_splits, win,
                            win_tiles, base_t, rem_t, r, L.waves, (int)grid.x, appends, q);
    else
      hipLaunchKernelGGL(kernel, grid, dim3(64u * L.waves), lds_bytes, L.stream, a, n_both, n_splits, win, win_tiles, base_t, rem_t, r,
                         L.waves, (int)grid.x, appends, q);
  };
#if INNERQ_INNER_JOIN
  const QuantArgs append = L.append ? *L.append : QuantArgs{};
#else
  const int append = 0;
#endif
  if (r <= 4) go(attention_inner_kernel<KB, VB, G, 1, ZK, ZV, !JOIN>, append);
  else if (!JOIN && L.waves == 1) go(attention_inner_kernel<KB, VB, G, 2, ZK, ZV, !JOIN>, append);
  else go(attention_inner_kernel<KB, VB, G, 2, ZK, ZV, false>, append);
  return hipGetLastError();
}

// 0: no value zero-point array; 1: read densely; 2: read only where a group is flagged
inline int value_zero_mode(const AttnArgs& a) { return a.v.zeros == nullptr ? 0 : (a.sparse_zeros ? 2 : 1); }

template <int KB, int VB, int G>
hipError_t launch_t(const AttnArgs& a, int n_both, int n_splits, const WindowSet& win, const Launch& L) {
  const bool zk = a.k.zeros != nullptr;
  const int zv = value_zero_mode(a);
  if (zk) {
    if (zv == 2) return launch_z<KB, VB, G, true, 2>(a, n_both, n_splits, win, L);
    if (zv == 1) return launch_z<KB, VB, G, true, 1>(a, n_both, n_splits, win, L);
    return launch_z<KB, VB, G, true, 0>(a, n_both, n_splits, win, L);
  }
  if (zv == 2) return launch_z<KB, VB, G, false, 2>(a, n_both, n_splits, win, L);
  if (zv == 1) return launch_z<KB, VB, G, false, 1>(a, n_both, n_splits, win, L);
  return launch_z<KB, VB, G, false, 0>(a, n_both, n_splits, win, L);
}

// Width pairs (keys, values) the fused kernel is built for: equal widths, and the paper's
// Hybrid / Small presets (3-bit keys, 2-bit values).
inline int width_pair(const AttnArgs& a) {
  if (a.bits == a.v_bits && a.bits >= 2 && a.bits <= 4) return a.bits - 2;   // 0, 1, 2
  if (a.bits == 3 && a.v_bits == 2) return 3;
  return -1;
}

}  // namespace

// The launch of this build (contiguous or paged store, one group size, joining or not).
hipError_t INNERQ_INNER_LAUNCH(const AttnArgs& a, int n_both, int n_splits, const WindowSet& win, const Launch& L) {
  constexpr int G = INNERQ_INNER_GROUP;
  if (a.group != G || (a.pages.table != nullptr) != kPagedStore || (a.join != nullptr) != JOIN) return hipErrorInvalidValue;
  switch (width_pair(a)) {
    case 0: return launch_t<2, 2, G>(a, n_both, n_splits, win, L);
    case 1: return launch_t<3, 3, G>(a, n_both, n_splits, win, L);
    case 2: return launch_t<4, 4, G>(a, n_both, n_splits, win, L);
    case 3: return launch_t<3, 2, G>(a, n_both, n_splits, win, L);
    default: return hipErrorInvalidValue;
  }
}

#if !INNERQ_PAGED_STORE && INNERQ_INNER_GROUP == 32 && !INNERQ_INNER_JOIN

bool attention_inner_supported(const AttnArgs& a) {
  const int r = a.n_q_heads / a.n_kv_heads;
  // offsets inside one (batch, kv-head) slab are 32-bit in the kernel
  return a.k.form == kPerToken && a.v.form == kPerChannel && width_pair(a) >= 0 && r <= 8 &&
         (a.group == 32 || a.group == 64) && a.capacity * D <= (1LL << 31);
}

std::atomic<int> g_inner_variant{0};

bool attention_inner_wants_f4(const AttnArgs& a) {
  return !a.pages.table && g_inner_variant.load(std::memory_order_relaxed) == 1 && attention_inner_f4_supported(a);
}

int attention_inner_waves_per_cu(const AttnArgs& a) {
  if (a.f4) return attention_inner_f4_waves_per_cu(a);
  return 8;                                            // two per SIMD, by the kernel's register bound
}

hipError_t launch_attention_inner(const AttnArgs& a, long long n_both, int n_splits, const WindowSet& win, int waves,
                                  const QuantArgs* append, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (!attention_inner_supported(a)) return hipErrorInvalidValue;
  if (a.f4) {
    if (a.join || append) return hipErrorInvalidValue;
    return launch_attention_inner_f4(a, n_both, n_splits, win, stream, ev_start, ev_stop);
  }
  const Launch L = {stream, ev_start, ev_stop, waves, append};
  const bool paged = a.pages.table != nullptr, wide = a.group != 32;
  const auto go = a.join ? (paged ? (wide ? launch_join_paged_g64 : launch_join_paged_g32) : (wide ? launch_join_g64 : launch_join_g32))
                         : (paged ? (wide ? launch_inner_paged_g64 : launch_inner_paged_g32) : (wide ? launch_inner_g64 : launch_inner_g32));
  return go(a, (int)n_both, n_splits, win, L);
}

#endif

}  // namespace innerq

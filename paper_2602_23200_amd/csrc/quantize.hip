// Quantise / pack kernels, window copies and key-norm calibration.
//
// This translation unit is compiled with -ffp-contract=off: the integer codes
// and the symmetric/asymmetric flag depend on every fp32 rounding, so each
// multiply, add, subtract and divide below is a separate IEEE operation
// (Section "Quantization Scheme", Eq. asym_quant; Figure "hybrid").
#include "innerq_dev.h"
#include "merge.h"
#include "quantize_rows.h"

namespace innerq {
namespace {

__global__ void __launch_bounds__(256) window_copy_kernel(QuantArgs a) {
  const QuantTensorJob j = pick_job(a, (int)blockIdx.y);
  window_copy(a, j, (long long)blockIdx.x * blockDim.x + threadIdx.x);
}

// (Registers: a long prompt waits for memory, and the copies into the windows in a short one for room beside the quantising work-groups.)
template <int G, int LANES, bool FAST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 32 ? 6 : 4))) quantize_kernel(QuantArgs a, long long copy_from) {
  // Thread indices below copy_from quantise evicted tokens, those from copy_from on write the
  // new tokens into the windows (one launch; only used when no new token lands in a ring slot
  // that this call still has to read).  copy_from < 0: no copy work in this launch.
  const QuantTensorJob j = pick_job(a, (int)blockIdx.y);
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (copy_from >= 0 && idx >= copy_from) {
    window_copy(a, j, idx - copy_from);
    return;
  }
  if (j.bits == 2) quantize_rows<G, 2, LANES, false, FAST>(a, j, idx);
  else if (j.bits == 3) quantize_rows<G, 3, LANES, false, false>(a, j, idx);
  else quantize_rows<G, 4, LANES, false, FAST && G == 64>(a, j, idx);
}

// The same launch with the log-sum-exp merge of an attention call riding along: the last
// work-groups (of job 0) merge four query heads each, or one where it has many partials (SHARED); the ones before them are
// quantize_kernel (the longer dependent chain, so it is dispatched first).  The two jobs touch
// disjoint memory (partials and output against store rows and window slots).
template <int G, bool SHARED>
__global__ void __launch_bounds__(256) quantize_merge_kernel(QuantArgs a, long long copy_from, AttnArgs m,
                                                             int quant_blocks) {
  if ((int)blockIdx.x >= quant_blocks) {
    const int wave = threadIdx.x >> 6;
    const long long bhq = SHARED ? (long long)blockIdx.x - quant_blocks : (long long)(blockIdx.x - quant_blocks) * 4 + wave;
    if (blockIdx.y == 0 && bhq < (long long)m.batch * m.n_q_heads) merge_head<SHARED ? 4 : 1>(m, bhq, wave, threadIdx.x & 63);
    return;
  }
  const QuantTensorJob j = pick_job(a, (int)blockIdx.y);
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (copy_from >= 0 && idx >= copy_from) {
    window_copy(a, j, idx - copy_from);
    return;
  }
  if (j.bits == 2) quantize_rows<G, 2, 8, true, false>(a, j, idx);
  else if (j.bits == 3) quantize_rows<G, 3, 8, true, false>(a, j, idx);
  else quantize_rows<G, 4, 8, true, false>(a, j, idx);
}

// Threads the quantise work of one tensor job needs.
template <int G, int LANES>
long long quantize_threads(const QuantArgs& a, const QuantTensorJob& j) {
  const long long BH = (long long)a.batch * a.n_kv_heads;
  const long long rows = j.row_end - j.row_begin;
  if (rows <= 0) return 0;
  if (j.form == kPerToken) return BH * rows * (kHeadDim / G) * LANES;
  if (j.form == kPerChannel) return BH * (rows / G) * kHeadDim * a.channel_lanes;
  return BH * rows * (kHeadDim / 8);
}

hipError_t window_copies(const QuantArgs& a, hipStream_t stream) {
  const long long n = copy_threads(a);
  if (n == 0) return hipSuccess;
  dim3 grid((unsigned)((n + 255) / 256), 2);
  window_copy_kernel<<<grid, 256, 0, stream>>>(a);
  return hipGetLastError();
}

template <int G, int LANES, bool FAST = false>
hipError_t launch_quantize_t(QuantArgs a, hipStream_t stream, const AttnArgs* merge) {
  // Per-channel groups of the form of eight lanes, spread over eight too: a lane's chain of a group is the longest of a short launch (us, one
  // lane -> eight: one value group of 8 heads G = 32 6.0 -> 3.8, G = 64 9.1 -> 4.2; steps at which one leaves its ring, 8 x 8 heads, 13.8 ->
  // 12.2, G = 64 16.7 -> 12.3; 3 bits, symmetric, 14.6 -> 13.2), up to 192 sequence-heads, 256 at G = 64 (steps with a spill, time of eight lanes over one:
  // 128 heads 0.92 to 0.95, 256 0.99 to 1.00, single shapes to 1.11, and 0.96 at G = 64; 512 1.08), 64 of groups of one variant, whose
  // chain is half as long (128: 18.2 -> 20.4).  Where the counts live on the device the launch holds a group of every sequence, and mostly
  // none leaves (us a step of sequences of 8 heads, G = 32, in which none, one and all have one leave: 16 of them 19.2 21.6 21.9 -> 19.6
  // 19.7 20.9, 24 25.7 28.0 29.4 -> 26.1 26.1 28.0, 32 30.5 33.8 33.9 -> 34.4 34.4 36.5, 8 16.6 19.8 19.9 -> 18.2 18.8 19.0): in the mean
  // over independent lengths 0.92 to 0.97 of the time from 16 sequences up to 192 heads, 1.02 to 1.10 from 256 heads on.
  const int mode = a.job[a.job[0].form == kPerChannel ? 0 : 1].mode;
  const long long bh = (long long)a.batch * a.n_kv_heads;
  const long long most_heads = mode != INNERQ_HYBRID ? 64 : G == 64 ? 256 : 192;
  const bool spread = bh <= most_heads && (!a.n_dev || (a.batch >= 16 && G == 32));
  a.channel_lanes = LANES == 8 && spread ? 8 : 1;
  const long long kthreads = quantize_threads<G, LANES>(a, a.job[0]), vthreads = quantize_threads<G, LANES>(a, a.job[1]);
  const long long threads = kthreads > vthreads ? kthreads : vthreads, cthreads = copy_threads(a);
  if (threads >= (1LL << 32)) return hipErrorInvalidValue;   // (device index arithmetic is 32-bit)
  // no ring slot shared by an evicted and a new token: one launch does both jobs
  const bool disjoint = !ring_slots_shared(a, a.job[0]) && !ring_slots_shared(a, a.job[1]);
  if (merge && disjoint) {
    // one launch: the quantise threads, the window-copy threads, then the merge blocks
    const long long qthreads = ((threads + 255) / 256) * 256;
    const long long heads = (long long)merge->batch * merge->n_q_heads;
    const bool shared = merge_is_shared(*merge);
    const int merge_blocks = (int)(shared ? heads : (heads + 3) / 4);
    const int quant_blocks = (int)((qthreads + cthreads + 255) / 256);
    dim3 grid((unsigned)(quant_blocks + merge_blocks), 2);
    if (shared) quantize_merge_kernel<G, true><<<grid, 256, 0, stream>>>(a, qthreads, *merge, quant_blocks);
    else quantize_merge_kernel<G, false><<<grid, 256, 0, stream>>>(a, qthreads, *merge, quant_blocks);
    return hipGetLastError();
  }
  if (merge) {
    const hipError_t e = launch_attention_merge(*merge, stream);
    if (e != hipSuccess) return e;
  }
  if (threads > 0 && disjoint) {
    const long long qthreads = ((threads + 255) / 256) * 256;
    dim3 grid((unsigned)((qthreads + cthreads + 255) / 256), 2);
    quantize_kernel<G, LANES, FAST><<<grid, 256, 0, stream>>>(a, qthreads);
    return hipGetLastError();
  }
  if (threads > 0) {
    dim3 grid((unsigned)((threads + 255) / 256), 2);
    quantize_kernel<G, LANES, FAST><<<grid, 256, 0, stream>>>(a, -1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return window_copies(a, stream);
}

// ---- key-norm calibration (Section "Per-channel Normalization of K") ----------------------

// The per-channel maxima (float bits) and the counts of finished work-groups live in the outputs, zeroed beforehand,
// until the last work-group turns the maxima into the factors.
struct AbsmaxPlan {
  const __half* k;
  long long n_tokens, tokens_per_block;
  int n_kv_heads, per_head;
  uint32_t blocks_per_head;           // work-groups of one kv head (over the batch)
  uint32_t* table;                    // [Hk][d], aliases inv_out
  uint32_t* done;                     // [Hk][d], aliases norm_out: entry 0 of a head counts its work-groups; entry 1 of head 0 the heads
                                      // (null where the two outputs share memory: the factors are then a launch of their own)
  float* norm_out;
  float* inv_out;
};

__global__ void calibrate_zero_kernel(uint32_t* table, uint32_t* done, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    table[i] = 0u;
    if (done) done[i] = 0u;
  }
}

// The factors from the maxima: one work-group, four threads a channel, every fourth head each; a thread reads its
// entries before it overwrites them.
constexpr int kCalibThreads = 512;
__device__ __forceinline__ void write_factors(const AbsmaxPlan& m) {
  constexpr int kShare = kCalibThreads / kHeadDim;
  const int c = threadIdx.x % kHeadDim, share = threadIdx.x / kHeadDim;
  auto entry = [&](int h) {
    return __uint_as_float(__hip_atomic_load(m.table + h * kHeadDim + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  __shared__ float part[kShare][kHeadDim];
  float all = 0.f;
  if (!m.per_head) {
    for (int h0 = share; h0 < m.n_kv_heads; h0 += 8 * kShare) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = entry(h0 + kShare * i < m.n_kv_heads ? h0 + kShare * i : h0);
#pragma unroll
      for (int i = 0; i < 8; ++i) all = fmaxf(all, v[i]);
    }
    part[share][c] = all;
  }
  __syncthreads();                                       // (every entry has been read)
  if (!m.per_head) {
#pragma unroll
    for (int i = 0; i < kShare; ++i) all = fmaxf(all, part[i][c]);
  }
  for (int h = share; h < m.n_kv_heads; h += kShare) {
    const float v = m.per_head ? entry(h) : all;
    const float n = v == 0.f ? 1.f : sqrtf(v);
    m.norm_out[h * kHeadDim + c] = n;
    m.inv_out[h * kHeadDim + c] = 1.0f / n;
  }
}

// max |K| per (kv head, channel): each work-group scans a slice of tokens of one (b, hk), eight rows a thread in
// flight, and folds its 128 channel maxima into the table with an unsigned atomic max on the float bits (monotone
// for non-negative floats).  The maxima of x and -x are packed fp16 ones, two channels an instruction, and pass a NaN
// over (a maximum of the bits would put one NaN key in the place of its channel's maximum); a plain read of the keys
// is what it takes (8 x 8 heads x 32k tokens: 82 us, 6.5 TB/s; 91 without the non-temporal loads; 101 before, one row a
// thread in flight).  Few, large work-groups: the atomics of a head meet in the same 128 entries, about 20 ns each, and
// so do the counts.
constexpr int kCalibRows = kCalibThreads / 16;   // token rows per pass of a work-group
constexpr int kCalibPasses = 8;                  // passes in flight
__global__ void __launch_bounds__(kCalibThreads) absmax_kernel(AbsmaxPlan m) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const long long bh = blockIdx.y;
  const int hk = (int)(blockIdx.y % (uint32_t)m.n_kv_heads);
  const int ch = threadIdx.x % 16, r = threadIdx.x / 16;
  const long long t0 = (long long)blockIdx.x * m.tokens_per_block;
  const long long t1 = t0 + m.tokens_per_block < m.n_tokens ? t0 + m.tokens_per_block : m.n_tokens;
  const u32x4* rows = reinterpret_cast<const u32x4*>(m.k + bh * m.n_tokens * kHeadDim + ch * 8);
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  f16x2 mx[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
  for (long long t = t0 + r; t < t1; t += kCalibRows * kCalibPasses) {
    u32x4 raw[kCalibPasses];
#pragma unroll
    for (int p = 0; p < kCalibPasses; ++p) {
      const long long tt = t + kCalibRows * p < t1 ? t + kCalibRows * p : t;      // (a row twice does not matter)
      raw[p] = __builtin_nontemporal_load(rows + tt * (kHeadDim / 8));
    }
#pragma unroll
    for (int p = 0; p < kCalibPasses; ++p) {
      const uint32_t w[4] = {raw[p].x, raw[p].y, raw[p].z, raw[p].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f16x2 x = __builtin_bit_cast(f16x2, w[e]);
        mx[e] = __builtin_elementwise_max(mx[e], __builtin_elementwise_max(x, -x));
      }
    }
  }
  __shared__ uint32_t red[kCalibRows][kHeadDim / 2];
#pragma unroll
  for (int e = 0; e < 4; ++e) red[r][ch * 4 + e] = __builtin_bit_cast(uint32_t, mx[e]) & 0x7fff7fffu;
  __syncthreads();
  // Table and counts are only ever touched by device-scope atomics (performed at the memory side, past the caches),
  // so no cache has to be written back or invalidated: a work-group counts itself done once its own atomic maxima
  // have RETURNED (their old values are consumed before the barrier), and the last one reads the table with atomic
  // loads.
  uint32_t seen = 0u;
  if (threadIdx.x < kHeadDim) {
    uint32_t v = 0u;
#pragma unroll
    for (int i = 0; i < kCalibRows; ++i) {
      const uint32_t w = red[i][threadIdx.x / 2], h = (threadIdx.x & 1u) ? w >> 16 : w & 0xffffu;
      v = v > h ? v : h;
    }
    seen = atomicMax(m.table + hk * kHeadDim + threadIdx.x, __float_as_uint(__half2float(__ushort_as_half((unsigned short)v))));
  }
  if (__syncthreads_or(seen == 0xffffffffu)) return;     // (never true: a maximum of |fp16| is finite)
  if (!m.done) return;                                   // (uniform)
  __shared__ uint32_t last;
  if (threadIdx.x == 0) {
    // (a count of one is not taken: every count is a memory round trip, the most of a short prompt's time; one head, 20
    // tokens 6.9 us with both)
    last = 0u;
    if (m.blocks_per_head == 1u || atomicAdd(m.done + hk * kHeadDim, 1u) == m.blocks_per_head - 1u)
      last = m.n_kv_heads == 1 || atomicAdd(m.done + 1, 1u) == (uint32_t)m.n_kv_heads - 1u;
  }
  __syncthreads();
  if (!last) return;
  write_factors(m);
}

__global__ void __launch_bounds__(kCalibThreads) factors_kernel(AbsmaxPlan m) { write_factors(m); }

}  // namespace

hipError_t launch_quantize(const QuantArgs& a, hipStream_t stream, const AttnArgs* merge) {
  for (int w = 0; w < 2; ++w)
    if (a.job[w].form != kFp16 && (a.job[w].bits < 2 || a.job[w].bits > 4)) return hipErrorInvalidValue;
  if (a.group != 32 && a.group != 64) return hipErrorInvalidValue;
  const AppendForm form = merge ? AppendForm::kLanes8 : append_form(a);
  if (form == AppendForm::kRingOwners || form == AppendForm::kRingOwnersPairs) return launch_quantize_owners(a, form == AppendForm::kRingOwnersPairs, stream);
  if (form == AppendForm::kLane) {
    // The shorter error sum for hybrid groups of 2 bits, and of 4 at G = 64, from 2 M groups on: 8 x 8 heads x 32k tokens (8.4 M) 259 us -> 250, 16k 131 -> 128, 8k
    // (1 M) the same; of the time without it 0.974 to 1.002 at G = 32 and 0.979 to 0.993 at G = 64, at 4 bits 1.01 to 1.04 and 0.98
    // to 1.00, at 3 bits 1.00 to 1.04.
    long long most = 0;
    bool gains = false;
    for (int w = 0; w < 2; ++w) {
      const long long groups = (long long)a.batch * a.n_kv_heads * (a.job[w].row_end - a.job[w].row_begin) * (kHeadDim / a.group);
      most = groups > most ? groups : most;
      gains = gains || (a.job[w].mode == INNERQ_HYBRID && (a.job[w].bits == 2 || (a.job[w].bits == 4 && a.group == 64)));
    }
    const bool fast = gains && most >= (1LL << 21);
    if (a.group == 32) return fast ? launch_quantize_t<32, 1, true>(a, stream, nullptr) : launch_quantize_t<32, 1>(a, stream, nullptr);
    return fast ? launch_quantize_t<64, 1, true>(a, stream, nullptr) : launch_quantize_t<64, 1>(a, stream, nullptr);
  }
  return a.group == 32 ? launch_quantize_t<32, 8>(a, stream, merge) : launch_quantize_t<64, 8>(a, stream, merge);
}

hipError_t launch_calibrate(const __half* k, int batch, int n_kv_heads, long long n_tokens, int per_head,
                            float* norm_out, float* inv_out, hipStream_t stream) {
  AbsmaxPlan m;
  m.k = k; m.n_tokens = n_tokens; m.n_kv_heads = n_kv_heads; m.per_head = per_head;
  m.table = reinterpret_cast<uint32_t*>(inv_out);
  m.norm_out = norm_out; m.inv_out = inv_out;
  const int n = n_kv_heads * kHeadDim;
  // counts and maxima in one place would spoil each other: a caller that wants one of the two vectors may pass its
  // buffer for both (1 / norm, written last, is what stays)
  const bool apart = norm_out + n <= inv_out || inv_out + n <= norm_out;
  m.done = apart ? reinterpret_cast<uint32_t*>(norm_out) : nullptr;
  calibrate_zero_kernel<<<(n + 255) / 256, 256, 0, stream>>>(m.table, m.done, n);   // (a kernel: safe inside a captured graph)
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // two work-groups per compute unit where there is that much to read, in slices of whole passes
  const long long step = kCalibRows * kCalibPasses, bh = (long long)batch * n_kv_heads;
  long long slices = 2LL * compute_units() / bh;
  slices = slices < 1 ? 1 : slices;
  m.tokens_per_block = ((n_tokens + slices - 1) / slices + step - 1) / step * step;
  dim3 grid((unsigned)((n_tokens + m.tokens_per_block - 1) / m.tokens_per_block), (unsigned)bh);
  m.blocks_per_head = grid.x * (unsigned)batch;
  absmax_kernel<<<grid, kCalibThreads, 0, stream>>>(m);
  e = hipGetLastError();
  if (e != hipSuccess || apart) return e;
  factors_kernel<<<1, kCalibThreads, 0, stream>>>(m);
  return hipGetLastError();
}

}  // namespace innerq

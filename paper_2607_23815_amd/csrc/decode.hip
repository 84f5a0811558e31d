// Paged decode attention for gfx950: the decode launch (an ordering kernel for long batches, the
// work items, and the merge of split partial results where sequences split). The work-item
// bodies are in decode_impl.h.
#include <math.h>

#include <mutex>

#include "decode_impl.h"
#include "decode_plan.h"

namespace pkv {
namespace {

constexpr int kWaves = 4;  // waves per workgroup of the merge kernel

// One wave per work item: a compute unit takes new work as soon as any wave ends (work items
// differ in length).
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_partial_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    int32_t max_blocks, dec::DecodeWork work, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale_log2, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    uint16_t* __restrict__ out, float* __restrict__ lse) {
  dec::decode_body<D>(q, k_cache, v_cache, block_tables, max_blocks, work, hq, hkv, num_blocks,
                      scale_log2, ws_o, ws_ml, out, lse, blockIdx.x);
}

// kParts waves per work item, merged inside the workgroup.
template <int D, int kParts>
__global__ __launch_bounds__(64 * kParts) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_group_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    int32_t max_blocks, dec::DecodeWork work, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale_log2, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    uint16_t* __restrict__ out, float* __restrict__ lse) {
  __shared__ __align__(16) dec::DecodeSmem<D, kParts> sm;
  dec::decode_group_body<D, kParts, kParts>(q, k_cache, v_cache, block_tables, max_blocks, work,
                                            hq, hkv, num_blocks, scale_log2, ws_o, ws_ml, out,
                                            lse, blockIdx.x, sm);
}

// One wave per (sequence, query head): combine the splits' partial (m_s, l_s, acc_s):
//   out = sum_s 2^(m_s - M) acc_s / sum_s 2^(m_s - M) l_s,   M = max_s m_s.
// Lane s of a round of 64 holds split s's maximum and weight sum, so a round waits for two
// loads and not for two per split; the outputs' loads do not depend on one another.
template <int D>
__global__ __launch_bounds__(256) void decode_merge_kernel(
    const float* __restrict__ ws_o, const float* __restrict__ ws_ml,
    const int32_t* __restrict__ seq_lens, int32_t num_seqs, int32_t hq, int32_t split_keys,
    int32_t max_splits, int32_t max_keys, uint16_t* __restrict__ out, float* __restrict__ lse) {
  constexpr int PER = D / 64;  // dims per lane
  const int64_t item = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (item >= (int64_t)num_seqs * hq) return;
  const int i = (int)(item / hq);
  const int len = min(seq_lens[i], max_keys);
  const int nsplit = (len + split_keys - 1) / split_keys;
  if (nsplit <= 1) return;  // written directly by the partial kernel
  const size_t base = (size_t)item * max_splits;
  float mmax = -INFINITY;
  for (int s = lane; s < nsplit; s += 64) mmax = fmaxf(mmax, ws_ml[(base + s) * 2]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mmax = fmaxf(mmax, __shfl_xor(mmax, o));
  const float m_sub = dec::finite_max(mmax);
  float den = 0.f;
  float o[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) o[e] = 0.f;
  for (int s0 = 0; s0 < nsplit; s0 += 64) {
    const int n = min(nsplit - s0, 64);
    float w = 0.f;
    if (lane < n) {
      w = fast_exp2(ws_ml[(base + s0 + lane) * 2] - m_sub);
      den += w * ws_ml[(base + s0 + lane) * 2 + 1];
    }
    const float* src = ws_o + (base + s0) * D + lane * PER;
    for (int s = 0; s < n; s += 8) add_partials<D>(src, w, s, n, o);
  }
#pragma unroll
  for (int k = 32; k >= 1; k >>= 1) den += __shfl_xor(den, k);
  const float inv = 1.f / den;
  uint16_t* dst = out + (size_t)item * D + lane * PER;
  if constexpr (PER == 2) {
    *reinterpret_cast<uint32_t*>(dst) = pack_bf16x2(o[0] * inv, o[1] * inv);
  } else {
    dst[0] = (uint16_t)(pack_bf16x2(o[0] * inv, 0.f) & 0xFFFFu);
  }
  if (lse != nullptr && lane == 0) lse[item] = (mmax + log2f(den)) * kLn2;
}

// Longest-first sequence order for a decode or prefill grid: work is dispatched in item
// order, so taking the longest sequences first keeps the launch from ending on a few long
// items. A sequence's length is lens[i], plus cu[i + 1] - cu[i] when cu is given (a prefill's
// cached and new tokens). Sequences are bucketed by length on a log scale (32 buckets per
// factor of two), counted, scanned in descending bucket order and scattered; order within a
// bucket follows the scatter's atomics and may differ from run to run, which the results do
// not depend on.
constexpr int kOrderBuckets = 2048;
constexpr int kOrderThreads = 1024;
__global__ __launch_bounds__(kOrderThreads) void decode_order_kernel(
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ cu, int32_t num_seqs,
    int32_t* __restrict__ order) {
  constexpr int kWavesO = kOrderThreads / 64;
  __shared__ int count[kOrderBuckets];
  __shared__ int base[kOrderBuckets];
  __shared__ int wsum[kWavesO];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  for (int b = t; b < kOrderBuckets; b += kOrderThreads) count[b] = 0;
  __syncthreads();
  auto bucket_of = [&](int i) {
    const int len = seq_lens[i] + (cu != nullptr ? cu[i + 1] - cu[i] : 0);
    if (len < 1) return 0;
    return min(1 + (int)(log2f((float)len) * 32.f), kOrderBuckets - 1);
  };
  for (int i = t; i < num_seqs; i += kOrderThreads) atomicAdd(&count[bucket_of(i)], 1);
  __syncthreads();
  // exclusive scan in descending bucket order: thread t owns descending positions 2t, 2t+1;
  // an inclusive scan within each wave (lane shuffles), then one over the waves' totals
  const int b0 = kOrderBuckets - 1 - 2 * t, b1 = b0 - 1;
  const int c0 = count[b0], c1 = count[b1];
  const int v = c0 + c1;
  int incl = v;
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  if (w == 0) {
    const int x = lane < kWavesO ? wsum[lane] : 0;
    int inc = x;
    for (int off = 1; off < kWavesO; off <<= 1) {
      const int u = __shfl_up(inc, off, 64);
      if (lane >= off) inc += u;
    }
    if (lane < kWavesO) wsum[lane] = inc - x;  // waves before this one
  }
  __syncthreads();
  const int excl = wsum[w] + incl - v;
  base[b0] = excl;
  base[b1] = excl + c0;
  __syncthreads();
  for (int i = t; i < num_seqs; i += kOrderThreads) order[atomicAdd(&base[bucket_of(i)], 1)] = i;
}


// KV bytes (at the host's longest length) from which a decode is ordered longest first: items of
// several shares, and items of one wave.
constexpr int64_t kOrderBytes = int64_t(512) << 20;
constexpr int64_t kOrderBytesOneWave = int64_t(400) << 20;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

// The allocation-free decode's workspace: one array per GPU, loaded with the code object and
// held until the process ends. Its device address comes from hipGetSymbolAddress, taken once
// per device with that device current; the array's name in host code is a host-side stand-in
// and never goes to a kernel or a copy.
static __device__ __align__(256) unsigned char scratch[kDecodeScratchBytes];

hipError_t decode_scratch(void** ptr) {
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return err;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

size_t decode_workspace_bytes(int32_t num_seqs, int32_t hq, int32_t hkv, int32_t head_dim,
                              int32_t max_seq_len) {
  const int32_t split = decode_split_keys(num_seqs, hkv, max_seq_len);
  const int64_t max_splits = (max_seq_len + split - 1) / split;
  // the sequence order, then (when sequences split) the partial results
  size_t bytes = order_bytes(num_seqs);
  if (max_splits > 1) bytes += (size_t)num_seqs * hq * max_splits * (head_dim + 2) * sizeof(float);
  return bytes;
}

DecodePlan decode_plan(const KvView& kv, int32_t hq, int32_t num_seqs, int32_t max_seq_len,
                       int32_t max_blocks, void* workspace) {
  DecodePlan p{decode_cut(num_seqs, kv.hkv, max_seq_len, max_blocks)};
  const int64_t groups = (int64_t)num_seqs * kv.hkv;
  // Longest first pays where not every wave is resident at once, or each stands alone for its
  // sequence's whole length, and the batch is long against the ordering launch (4.5 us): 256
  // sequences of 256-4096 keys 383 us against 399, 256 of 400-1200 154 against 156, but 200 of
  // 50-300 30 against 27. One wave per item, ordered against not: 2048 pairs of 1-513 keys 57.5
  // us against 59.2, 3072 of 1-300 (the bytes of 450 MB) 53.9 against 55.7, 3200 of 64 dims and
  // 1-300 keys (235 MB) 28.8 against 27.0.
  // Up to 64 sequences the waves find the order themselves (48 of 256-4096 keys, 64/8 heads:
  // 79.1 us against 81.2; 60 of 400-8000, 8/8 heads 176.4 against 177.6; short batches, which
  // take no order, would lose 2-3 us by it).
  const int64_t bytes = groups * max_seq_len * kv.head_dim * 4;
  const bool longest_first =
      p.parts == 1 ? bytes >= kOrderBytesOneWave
                   : p.items * p.parts > kWaveSlots && bytes >= kOrderBytes;
  p.by_rank = longest_first && num_seqs <= kRankSeqs;
  p.ordered = longest_first && !p.by_rank;
  p.order = static_cast<int32_t*>(workspace);
  p.ws_o = nullptr;
  p.ws_ml = nullptr;
  if (p.max_splits > 1) {
    p.ws_o = reinterpret_cast<float*>(static_cast<char*>(workspace) + order_bytes(num_seqs));
    p.ws_ml = p.ws_o + (size_t)num_seqs * hq * p.max_splits * kv.head_dim;
  }
  return p;
}

size_t order_bytes(int32_t num_seqs) {
  return ((size_t)num_seqs * sizeof(int32_t) + 255) / 256 * 256;
}

hipError_t launch_seq_order(const int32_t* lens, const int32_t* cu, int32_t num_seqs,
                            int32_t* order, hipStream_t stream) {
  hipLaunchKernelGGL(decode_order_kernel, dim3(1), dim3(kOrderThreads), 0, stream, lens, cu,
                     num_seqs, order);
  return hipGetLastError();
}

hipError_t launch_decode_order(const DecodePlan& p, const int32_t* seq_lens, int32_t num_seqs,
                               hipStream_t stream) {
  if (!p.ordered) return hipSuccess;
  return launch_seq_order(seq_lens, nullptr, num_seqs, p.order, stream);
}

hipError_t launch_decode_merge(const KvView& kv, const DecodePlan& p, int32_t hq,
                               const int32_t* seq_lens, int32_t num_seqs, uint16_t* out,
                               float* lse, hipStream_t stream) {
  if (p.max_splits <= 1) return hipSuccess;
  const int64_t rows = (int64_t)num_seqs * hq;
  const dim3 mgrid((unsigned)((rows + kWaves - 1) / kWaves));
  if (kv.head_dim == 128)
    hipLaunchKernelGGL(decode_merge_kernel<128>, mgrid, dim3(256), 0, stream, p.ws_o, p.ws_ml,
                       seq_lens, num_seqs, hq, p.split, p.max_splits, p.max_keys, out, lse);
  else
    hipLaunchKernelGGL(decode_merge_kernel<64>, mgrid, dim3(256), 0, stream, p.ws_o, p.ws_ml,
                       seq_lens, num_seqs, hq, p.split, p.max_splits, p.max_keys, out, lse);
  return hipGetLastError();
}

hipError_t launch_decode(const KvView& kv, const uint16_t* q, int32_t hq,
                         const int32_t* block_tables, int32_t max_blocks,
                         const int32_t* seq_lens, int32_t num_seqs, int32_t max_seq_len,
                         float scale, uint16_t* out, float* lse, void* workspace,
                         hipStream_t stream) {
  const DecodePlan p = decode_plan(kv, hq, num_seqs, max_seq_len, max_blocks, workspace);
  if (p.items * 64 * p.parts > kGridThreads) return hipErrorInvalidValue;
  const dim3 grid((unsigned)p.items);
  const float scale_log2 = scale * kLog2e;
  hipError_t err = launch_decode_order(p, seq_lens, num_seqs, stream);
  if (err != hipSuccess) return err;
  const bool wide = kv.head_dim == 128;
  auto* kern = p.parts == 1 ? (wide ? decode_partial_kernel<128> : decode_partial_kernel<64>)
             : p.parts == 4 ? (wide ? decode_group_kernel<128, 4> : decode_group_kernel<64, 4>)
                            : (wide ? decode_group_kernel<128, 8> : decode_group_kernel<64, 8>);
  hipLaunchKernelGGL(kern, grid, dim3(64 * p.parts), 0, stream, q, kv.k, kv.v, block_tables,
                     max_blocks, decode_work(p, seq_lens, num_seqs), hq, kv.hkv, kv.num_blocks,
                     scale_log2, p.ws_o, p.ws_ml, out, lse);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_decode_merge(kv, p, hq, seq_lens, num_seqs, out, lse, stream);
}

}  // namespace pkv

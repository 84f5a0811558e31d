// Whole-block copies for copy-on-write, for gfx950. A block's K region for all kv heads is one
// contiguous span of hkv * D * 16 elements of the K cache ([block][hkv][D/8][16][8]), and
// likewise its V region ([block][hkv][D][16]), so a copy is a plain 16-byte vector copy,
// coalesced across the workgroup.
#include <algorithm>

#include "device_utils.h"
#include "launch.h"

namespace pkv {
namespace {

// Workgroup (k, which, part) copies one part (kUnroll x 256 chunks) of the K (which = 0) or V
// (which = 1) region of block pairs[2k] to block pairs[2k+1]; a pair naming a block outside the
// pool is skipped. A copy waits for memory, not for bandwidth: a thread has all its loads in
// flight before its first store (the two regions never overlap), and a region is cut into
// parts so that a few pairs still spread over the chip. 255 pairs of 32 KB regions and the
// append that follows, from cold caches: 33.6 us with one workgroup per region (eight loads
// and stores, one after another), 31.5 with two loads per thread; one, two and four are equal
// within 1%, eight are slower (34.6).
constexpr int kUnroll = 2;
constexpr int kCopyThreads = 256;
constexpr int64_t kMaxParts = 65535;  // (a grid's z)
template <bool kMany>  // regions of more parts than the grid has: a workgroup copies several
__global__ __launch_bounds__(kCopyThreads) void copy_blocks_kernel(
    uint16_t* __restrict__ k_cache, uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ pairs, int32_t num_blocks, int64_t span) {
  const int32_t src = pairs[2 * blockIdx.x];
  const int32_t dst = pairs[2 * blockIdx.x + 1];
  if (src < 0 || src >= num_blocks || dst < 0 || dst >= num_blocks || src == dst) return;
  uint16_t* base = blockIdx.y == 0 ? k_cache : v_cache;
  const u32x4* from = reinterpret_cast<const u32x4*>(base + (size_t)src * span);
  u32x4* to = reinterpret_cast<u32x4*>(base + (size_t)dst * span);
  const int64_t n = span / 8;  // 16-byte chunks
  constexpr int64_t kPart = kUnroll * kCopyThreads;
  int64_t c0 = blockIdx.z * kPart + threadIdx.x;
  do {
    u32x4 v[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k)
      if (c0 + k * kCopyThreads < n) v[k] = from[c0 + k * kCopyThreads];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k)
      if (c0 + k * kCopyThreads < n) to[c0 + k * kCopyThreads] = v[k];
    c0 += gridDim.z * kPart;
  } while (kMany && c0 < n);
}

}  // namespace

hipError_t launch_copy_blocks(const KvView& kv, const int32_t* pairs, int32_t num_pairs,
                              hipStream_t stream) {
  const int64_t span = (int64_t)kv.hkv * kv.head_dim * kBlockSize;
  const int64_t part = (int64_t)kUnroll * kCopyThreads * 8;  // elements
  const int64_t parts = (span + part - 1) / part;
  const dim3 grid((unsigned)num_pairs, 2, (unsigned)std::min(parts, kMaxParts));
  auto* kern = parts > kMaxParts ? copy_blocks_kernel<true> : copy_blocks_kernel<false>;
  hipLaunchKernelGGL(kern, grid, dim3(kCopyThreads), 0, stream, kv.k, kv.v, pairs,
                     kv.num_blocks, span);
  return hipGetLastError();
}

}  // namespace pkv

// Mixed prefill + decode attention for gfx950: one fused launch in which some workgroups run
// prefill work items (the matrix-core-bound body of prefill_impl.h) and others decode work (the
// HBM-bound bodies of decode_impl.h: one item shared by the four waves, or four one-wave items,
// as the decode plan says), so that each compute unit overlaps the two kinds of work instead of
// running them one launch after the other.
//
// Workgroup b runs on XCD b % 8. Each XCD's list of positions b / 8 is dealt between prefill
// and decode workgroups in proportion to their counts, spread evenly along the list (few and
// long decode items go first: kFrontItems); a prefill workgroup keeps the XCD its index would
// have in a prefill-only launch (its index has the same residue mod 8), so the (sequence, kv
// head) groups keep their XCD and L2. The decode items follow the longest-first order of the
// decode launch, and the results are bit-identical to a prefill launch followed by a decode
// launch.
#include <algorithm>

#include "decode_plan.h"
#include "launch.h"
#include "prefill_impl.h"

namespace pkv {
namespace {

constexpr int kDecodePerWg = pre::kThreads / 64;  // one-wave decode items per workgroup

// kParts: shares per decode item (1: four one-wave items per workgroup)
template <int D, int kParts>
__global__ __attribute__((amdgpu_flat_work_group_size(pre::kThreads, pre::kThreads),
                          amdgpu_waves_per_eu(2, 2)))
void mixed_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
                  const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
                  int32_t max_blocks, const int32_t* __restrict__ cached_lens,
                  const int32_t* __restrict__ cu_new_lens, int32_t num_seqs, int32_t hq,
                  int32_t hkv, int32_t num_blocks, int32_t qtiles, float scale_log2,
                  uint16_t* __restrict__ out, float* __restrict__ lse,
                  const uint16_t* __restrict__ dq, const int32_t* __restrict__ d_tables,
                  int32_t d_max_blocks, dec::DecodeWork work, float* __restrict__ ws_o,
                  float* __restrict__ ws_ml, uint16_t* __restrict__ d_out,
                  float* __restrict__ d_lse, int32_t spread, int32_t d8, int64_t d_items) {
  __shared__ __align__(16) union {
    pre::PrefillSmem<D> prefill;
    dec::DecodeSmem<D, kParts> decode;
  } sm;
  const unsigned x = blockIdx.x & 7;
  const unsigned pos = blockIdx.x >> 3;
  // decode workgroups before position pos, and up to and including it: the XCD's d8 of them spread
  // evenly over its first `spread` positions
  const int64_t before = min((int64_t)pos * d8 / spread, (int64_t)d8);
  const int64_t upto = min(((int64_t)pos + 1) * d8 / spread, (int64_t)d8);
  if (upto > before) {
    const int64_t wg = (int64_t)before * 8 + x;
    if constexpr (kParts == 1) {
      // The wave index goes through readfirstlane: without it every load of the item sits in a loop
      // over lanes, as the compiler cannot tell that a wave's lanes share it. 256 sequences of
      // 1-500 keys beside 64 prefilling ones, 64/8 heads, 345 us with it and 353 without, 256
      // beside 8, 8/8 heads of 64 dims, 50.2 and 52.2; where the decode is most of the launch the
      // loops hold its waves back to the prefill's good: 384 of 1-1000 beside 8, 32/8 heads, 196
      // and 193.
      const int64_t item =
          wg * kDecodePerWg + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
      if (item >= d_items) return;
      dec::decode_body<D>(dq, k_cache, v_cache, d_tables, d_max_blocks, work, hq, hkv,
                          num_blocks, scale_log2, ws_o, ws_ml, d_out, d_lse, item);
    } else {
      if (wg >= d_items) return;
      dec::decode_group_body<D, kParts, kDecodePerWg>(
          dq, k_cache, v_cache, d_tables, d_max_blocks, work, hq, hkv, num_blocks, scale_log2,
          ws_o, ws_ml, d_out, d_lse, wg, sm.decode);
    }
  } else {
    pre::prefill_body<D>(q, k_cache, v_cache, block_tables, max_blocks, cached_lens,
                         cu_new_lens, num_seqs, hq, hkv, num_blocks, qtiles, scale_log2, out,
                         lse, (unsigned)((pos - before) * 8 + x), sm.prefill);
  }
}

// Eight shares run on four waves here, two rounds each, so an item takes about twice as long as in
// a decode launch. Where a launch has no more of them than compute units and they are long, one that
// starts late in the list outlasts the prefill: such decode workgroups stand at the list's front. 32
// sequences of 800-7000 keys beside 8 prefilling of 64-256 tokens, 32/8 heads: 162 us spread evenly,
// 120 in front (131 as two launches); 32 of 256-4096 beside 2, 64/8 heads, 95 and 77. Over 420 launches
// of 16-504 pairs, 2-64 prefilling sequences and contexts of 2-16k the front is 14% faster within this
// line; outside it is up to 17% slower (16 of 256-4096 beside 2, 32/8 heads: 37 and 44), as the
// prefill then has its share of every compute unit only after the decode.
constexpr int64_t kFrontItems = 256;
constexpr int64_t kFrontBytes = 3 << 19;  // K and V of an item: 3072 keys of 128 dims

}  // namespace

hipError_t launch_mixed(const KvView& kv, int32_t hq, float scale, const uint16_t* q,
                        const int32_t* block_tables, int32_t max_blocks,
                        const int32_t* cached_lens, const int32_t* cu_new_lens, int32_t num_seqs,
                        int32_t max_new_len, uint16_t* out, float* lse, const uint16_t* dq,
                        const int32_t* d_block_tables, int32_t d_max_blocks,
                        const int32_t* seq_lens, int32_t d_num_seqs, int32_t max_seq_len,
                        uint16_t* d_out, float* d_lse, void* workspace, hipStream_t stream) {
  const pre::PrefillGrid pg = pre::prefill_grid(hq, kv.hkv, num_seqs, max_new_len);
  const DecodePlan dp = decode_plan(kv, hq, d_num_seqs, max_seq_len, d_max_blocks, workspace);
  const int64_t d_wgs =
      dp.parts == 1 ? (dp.items + kDecodePerWg - 1) / kDecodePerWg : dp.items;
  const int64_t p8 = pg.items / 8;  // a multiple of 8 by construction
  const int64_t d8 = (d_wgs + 7) / 8;
  if (8 * (p8 + d8) * pre::kThreads > kGridThreads) {
    // A workgroup per item of several shares takes more of the grid than a wave per item: what
    // does not fit any more goes out as the two launches, whose results are the same.
    if (dp.parts == 1) return hipErrorInvalidValue;
    const hipError_t err =
        launch_prefill(kv, q, hq, block_tables, max_blocks, cached_lens, cu_new_lens, num_seqs, 0,
                       max_new_len, 0, scale, out, lse, nullptr, stream);
    if (err != hipSuccess) return err;
    return launch_decode(kv, dq, hq, d_block_tables, d_max_blocks, seq_lens, d_num_seqs,
                         max_seq_len, scale, d_out, d_lse, workspace, stream);
  }
  const dim3 grid((unsigned)(8 * (p8 + d8)));
  const float scale_log2 = scale * kLog2e;
  hipError_t err = launch_decode_order(dp, seq_lens, d_num_seqs, stream);
  if (err != hipSuccess) return err;
  const int64_t item_bytes = (int64_t)std::min(dp.split, max_seq_len) * kv.head_dim * 4;
  const bool front = dp.parts == 8 && dp.items <= kFrontItems && item_bytes >= kFrontBytes;
  const int64_t spread = front ? d8 : p8 + d8;
  const bool wide = kv.head_dim == 128;
  auto* kern = dp.parts == 1 ? (wide ? mixed_kernel<128, 1> : mixed_kernel<64, 1>)
             : dp.parts == 4 ? (wide ? mixed_kernel<128, 4> : mixed_kernel<64, 4>)
                             : (wide ? mixed_kernel<128, 8> : mixed_kernel<64, 8>);
  hipLaunchKernelGGL(kern, grid, dim3(pre::kThreads), 0, stream, q, kv.k, kv.v, block_tables,
                     max_blocks, cached_lens, cu_new_lens, num_seqs, hq, kv.hkv, kv.num_blocks,
                     (int32_t)pg.qtiles, scale_log2, out, lse, dq, d_block_tables, d_max_blocks,
                     decode_work(dp, seq_lens, d_num_seqs), dp.ws_o, dp.ws_ml, d_out, d_lse,
                     (int32_t)spread, (int32_t)d8, dp.items);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_decode_merge(kv, dp, hq, seq_lens, d_num_seqs, d_out, d_lse, stream);
}

}  // namespace pkv

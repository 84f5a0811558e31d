// How a decode call is cut into work items: host arithmetic on the call's sizes alone (no HIP,
// so that it can be compiled and checked without a GPU).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace pkv {

// Waves of the decode kernels that the chip holds at once (two on each of 256 x 4 SIMDs).
constexpr int64_t kWaveSlots = 2048;
constexpr int64_t kComputeUnits = 256;
// Threads that a launch's grid can hold.
constexpr int64_t kGridThreads = UINT32_MAX;
// Work items past which a launch stays at one wave each: items of eight waves would run into
// kGridThreads at 2^23 of them, where one wave each runs into it at 2^26.
constexpr int64_t kMaxWideItems = int64_t(1) << 20;

struct DecodeCut {
  int32_t split, max_splits;  // keys per split (a multiple of 32), splits of the longest sequence
  int32_t parts;              // waves' shares per work item (1: one wave is the item)
  int32_t max_keys;           // lengths are cut to it
  int64_t items;              // (sequence, kv head, split) work items
};

// The splits a call's workspace has room for: of 4096 keys, halved while a grid of one-wave items
// would hold fewer than 2048 waves. A function of the call's sizes only, so a given call always
// needs the same workspace. The cut below never makes more of them, mostly fewer; the size stays
// what callers have laid out for, and what decides the calls the fixed scratch takes.
inline int32_t decode_split_keys(int32_t num_seqs, int32_t hkv, int32_t max_seq_len) {
  int32_t split = 4096;
  while (split > 64) {
    const int64_t waves =
        (int64_t)num_seqs * hkv * ((max_seq_len + split - 1) / split);
    if (waves >= 2048) break;
    split /= 2;
  }
  return split;
}

// max_seq_len <= max_blocks * 16 (the length of a block table's row in keys).
inline DecodeCut decode_cut(int32_t num_seqs, int32_t hkv, int32_t max_seq_len,
                            int32_t max_blocks) {
  DecodeCut p;
  // What the workspace holds.
  const int32_t base_split = decode_split_keys(num_seqs, hkv, max_seq_len);
  const int64_t keys = ((int64_t)max_seq_len + base_split - 1) / base_split * base_split;
  // (sequence, kv head) pairs: the least number of work items
  const int64_t groups = (int64_t)num_seqs * hkv;
  // Shares per item. Cutting an item between the waves of one workgroup costs one LDS merge
  // and no launch, and evens out the waves' lengths, so four shares are the rule. Eight pay
  // where four would leave wave slots empty and some sequences are long enough to run on
  // alone (48 sequences of 256-4096 keys, 64/8 heads: 84 us against 104); below 2048 keys they
  // never do (32/8 heads, 1, 16 and 64 sequences of 800-1000 keys: 10.4 us against 9.6, 13.3
  // against 12.6, 48.5 against 46.3; of 200-256 keys 8.4 = 8.4, 8.2 = 8.2, 16.7 against 12.9).
  // One wave per item is left where the pairs alone fill the chip and the sequences are short:
  // more pairs are more rounds of waves, which even out by themselves, so the line rises with
  // them. One wave against four, of 1-n keys: 2048 pairs of 128 dims at n = 513 57.5 us against
  // 57.6, at 700 74.8 against 73.4; 3072 at 513 83.2 against 87.6, at 1000 149.2 against 149.8,
  // at 1499 216.0 against 213.7; 4096 at 513 104.2 against 109.4, at 1200 222.1 against 224.5;
  // 4096 of 64 dims at 513 54.8 against 61.5, at 1000 97.6 against 98.5, at 1499 142.5 against
  // 140.5; and beside a prefill of 8 sequences 3072 of 128 dims at 1000 196 against 207.
  if (groups >= kWaveSlots && (int64_t)max_seq_len * 3 <= groups)
    p.parts = 1;
  else if (groups < kWaveSlots / 4 && max_seq_len >= 2048)
    p.parts = 8;
  else
    p.parts = 4;
  for (;;) {
    // Splits across workgroups cost partial results and a merge launch (about 4 us), so they
    // are made only while the items leave the chip without enough loads in flight (waves aimed
    // at: `target`), and of at least 1024 keys (4 sequences of 24-32k keys, 32/8 heads: 87 us,
    // at 1.6 times fewer or 2 times more splits 92-104; one sequence of 800 keys with its
    // append: 12.1 us of kernels unsplit, 13.5 in two splits). At most 16384 keys, so that one
    // long sequence does not outlast the rest. A workgroup of eight shares fills a compute unit:
    // where every pair is one item and they come to a round and a bit, long sequences of nearly
    // the same length leave most units idle in the last round. So sequences above 16384 keys are
    // cut at 8192 there (17 of 20000-32000 keys, 8 heads of 128 dims: 448 us at 16384, 374 at
    // 8192; 62 of 6700-21400: 703 and 612), and where pairs are few more than units those above
    // 8192 at 4096 (33 of 15000-16000: 471 and 389). Lengths that balance by themselves pay for
    // it (17 of 1000-32000: 223 and 241; 33 of 4000-16000: 254 and 307), though less than one wave
    // per item did (294, 323). Up to 8192 keys they would pay more than the others gain (33 of
    // 7000-8000: 230 unsplit, 213 at 4096; of 4000-8000 156 and 189).
    const int64_t target = p.parts == 1 ? 1 : p.parts == 8 ? kWaveSlots : kWaveSlots / 2;
    const int64_t want = std::max<int64_t>(1, target / (groups * p.parts));
    int64_t split = std::max<int64_t>((keys + want - 1) / want, 1024);
    const bool few_over = groups > kComputeUnits && groups <= kComputeUnits * 5 / 4;
    const int64_t cap = p.parts != 8 || want > 1   ? 16384
                        : keys > 16384             ? 8192
                        : few_over && keys > 8192  ? 4096
                                                   : 16384;
    split = std::max<int64_t>(std::min<int64_t>(split, cap), base_split);
    const int64_t unit = 32 * p.parts;
    p.split = (int32_t)((split + unit - 1) / unit * unit);
    // Lengths are cut to the keys above and to the table's row: then every split of a cut length
    // starts inside the row (split sizes need not be multiples of base_split), so none is empty.
    p.max_keys = (int32_t)std::min<int64_t>({keys, (int64_t)max_blocks * 16, INT32_MAX});
    p.max_splits = (int32_t)(((int64_t)p.max_keys + p.split - 1) / p.split);
    p.items = groups * p.max_splits;
    if (p.parts == 1 || p.items < kMaxWideItems) break;
    p.parts = 1;
  }
  return p;
}

}  // namespace pkv

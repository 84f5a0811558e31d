// Paged decode attention for gfx950 (the per-wave work-item body, shared by the decode
// launch and the mixed prefill + decode launch): one query token per sequence over its whole cached
// context, split along the key axis ("split-K") so that every compute unit streams KV at the
// HBM rate, followed by a merge of the splits' partial results by their log-sum-exp weights.
//
// Work item = (sequence, kv head, split). Its keys are shared out among the waves of one
// workgroup (or one wave takes them all: see decode_cut and kLoneKeys for when), each wave streams
// its share on its own, without barriers, and the shares' results meet in LDS at the end. Cutting
// inside the workgroup needs no partial results in memory and no merge launch, so splits
// across workgroups are left to batches too small to fill the chip without them. HBM
// bandwidth bounds a large batch (512 sequences of 512-2048 keys: 5.9 TB/s), the chain of
// dependent loads (length, table, first K/V) and the launches a small one (one sequence of 800
// keys with its append: 17.2 us of kernels as ordering + 64-key splits + merge launches, 12.1 us
// as one). A long batch is taken longest first (past 64 sequences an ordering kernel runs before
// the launch, up to 64 every wave ranks the lengths for itself).
// A wave streams 32 keys (two 16-token blocks) at a time straight from HBM into the
// matrix-core operands:
//   scores  S^T[32 keys][16 cols] = K[keys][D] . Q^T[D][cols]      (v_mfma 16x16x32 bf16)
//   values  O^T[D][16 cols]      += V^T[D][32 keys] . P^T[keys][cols]
// The columns are the g = Hq/Hkv query heads that share the kv head (g <= 16; unused columns
// carry zero queries), so every KV byte is read once per kv head, never once per query head.
// Both products take 16-byte K loads and 8-byte V loads that are contiguous across the wave:
// the K pool slab is chunk-major ([D/8][16 slots][8]), so lane (slot s, chunk group q) of
// load kk reads chunk q + 4kk of slot s and one instruction covers 1 KB contiguous; the V pool
// slab is dim-major ([D][16 slots]), so lanes read 4 consecutive slots of one dim.
// The online softmax runs in the base-2 domain (scale * log2 e folded in fp32); per-column
// max and sum are combined across the four lane groups holding a column with cross-lane
// shuffles. Keys outside the sequence (tail slots of its last block, which may hold any bits,
// NaN included) are removed by selection -- scores to -inf and V operands to zero -- never by
// multiplying by a zero weight.
// The cuts depend on the call's sizes and each sequence's length only, so results are
// bit-identical from run to run and independent of where blocks sit in the pool.
#pragma once

#include <math.h>

#include "device_utils.h"

namespace pkv {
namespace dec {

__device__ __forceinline__ float wave_max16(float x) {
  // max over the four lanes l, l^16, l^32, l^48 (the lane groups holding one column)
  x = fmaxf(x, __shfl_xor(x, 16));
  x = fmaxf(x, __shfl_xor(x, 32));
  return x;
}
__device__ __forceinline__ float wave_sum16(float x) {
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}

// The maximum to subtract: a range whose scores are all -inf weighs nothing instead of
// 2^(-inf + inf) = NaN, so that cutting a sequence's keys into more ranges brings in no NaN.
__device__ __forceinline__ float finite_max(float m) { return m == -INFINITY ? 0.f : m; }

// zero the 16-bit lanes of a 4-element V fragment whose key index (base + e) >= nvalid
__device__ __forceinline__ u32x2 mask_v4(u32x2 v, int base, int nvalid) {
  uint32_t w0 = v[0], w1 = v[1];
  if (base + 0 >= nvalid) w0 &= 0xFFFF0000u;
  if (base + 1 >= nvalid) w0 &= 0x0000FFFFu;
  if (base + 2 >= nvalid) w1 &= 0xFFFF0000u;
  if (base + 3 >= nvalid) w1 &= 0x0000FFFFu;
  u32x2 r = {w0, w1};
  return r;
}

// K and V operands of one 32-key step (two blocks) of one wave, straight from HBM:
// K: lane (slot col, group grp) holds chunk grp + 4 kk of slot col of each block;
// V: lane holds slots 4 grp .. 4 grp + 3 of dim row 16 db + col of each block.
template <int D>
struct DecodeFrag {
  u32x4 k[2][D / 32];
  u32x2 v[2][D / 16];
};

template <int D>
__device__ __forceinline__ void decode_load(DecodeFrag<D>& f, const uint16_t* __restrict__ k_cache,
                                            const uint16_t* __restrict__ v_cache, size_t b0_off,
                                            size_t b1_off, int col, int grp) {
  // wave-uniform slab bases plus 32-bit per-lane byte offsets
  constexpr int SLAB_BYTES = D * kBlockSize * 2;
  const uint16_t* k0 = k_cache + b0_off;
  const uint16_t* k1 = k_cache + b1_off;
  const uint16_t* v0 = v_cache + b0_off;
  const uint16_t* v1 = v_cache + b1_off;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {
    const int o = ((grp + 4 * kk) * kBlockSize + col) * 16;
    f.k[0][kk] = buf_ld16(k0, SLAB_BYTES, o);
    f.k[1][kk] = buf_ld16(k1, SLAB_BYTES, o);
  }
#pragma unroll
  for (int db = 0; db < D / 16; ++db) {
    const int o = ((db * 16 + col) * kBlockSize + 4 * grp) * 2;
    f.v[0][db] = buf_ld8(v0, SLAB_BYTES, o);
    f.v[1][db] = buf_ld8(v1, SLAB_BYTES, o);
  }
}

// One wave's share of a work item: the keys [k0, k1) of a sequence (k0 a multiple of 16), for
// the columns of kv head kvh. Leaves the unnormalised output (lane (col, grp) holds dims
// 16 db + 4 grp + 0..3 of column col), the running maximum (base 2) and the lane's part of the
// weight sum. The range is not empty.
template <int D>
__device__ __forceinline__ void decode_range(
    const bf16x8 (&qf)[D / 32], const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ table, int32_t max_blocks,
    int32_t hkv, int32_t num_blocks, const int kvh, const int k0, const int k1,
    const float scale_log2, f32x4 (&acc_out)[D / 16], float& m_out, float& lpart_out) {
  constexpr int KK = D / 32;   // k-steps of the score product
  constexpr int DB = D / 16;   // 16-dim blocks of the value product
  constexpr int SLAB = D * kBlockSize;
  const int lane = threadIdx.x & 63;
  const int col = lane & 15;
  const int grp = lane >> 4;

  // The range's blocks in per-lane register tables of 64 entries: chunk c holds, in lane l,
  // the pool offset of the range's block 64 c + l, or of pool block 0 (a stand-in that is
  // read but masked) for blocks past the range, past the table or out of the pool. Two
  // chunks are live (the current one and the next), so every load below is unconditional
  // and a step's 24 loads issue back to back and overlap the previous step.
  const int b_first = k0 / kBlockSize;
  const int nblk = (k1 - k0 + kBlockSize - 1) / kBlockSize;
  // (the load and the check are separate steps, so that the first two chunks' loads are both
  // in flight before either is checked)
  auto raw_chunk = [&](int c) -> int {
    const int r = 64 * c + lane;
    const int b = b_first + r;
    return (r < nblk && b < max_blocks) ? table[b] : 0;
  };
  auto checked = [&](int e) -> int { return (e < 0 || e >= num_blocks) ? 0 : e; };
  auto load_chunk = [&](int c) -> int { return checked(raw_chunk(c)); };
  int chunk = 0;
  const int raw0 = raw_chunk(0), raw1 = raw_chunk(1);
  int tab = checked(raw0);
  int tab_next = checked(raw1);
  const size_t head_off = (size_t)kvh * SLAB;
  // block b (0 <= b < 128) counted from the start of the current chunk
  auto block_off = [&](int b) -> size_t {
    const int e = b < 64 ? __builtin_amdgcn_readlane(tab, b)
                         : __builtin_amdgcn_readlane(tab_next, b - 64);
    return (size_t)e * hkv * SLAB + head_off;
  };

  // Locals, copied out at the end: accumulated through the caller's references, the loop takes
  // 248 registers of a wave instead of 192, and the fused launch spills (2 registers with four
  // shares, 8 with eight).
  f32x4 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY;
  float lpart = 0.f;

  auto compute = [&](const DecodeFrag<D>& f, int t0) {
    const int nvalid = min(32, k1 - t0);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      s0 = mfma16(as_bf16x8(f.k[0][kk]), qf[kk], s0);
      s1 = mfma16(as_bf16x8(f.k[1][kk]), qf[kk], s1);
    }
    // lane holds keys 4*grp + r (block 0) and 16 + 4*grp + r (block 1) of column col
    float sv[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sv[r] = s0[r] * scale_log2;
      sv[4 + r] = s1[r] * scale_log2;
    }
    if (nvalid < 32) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sv[r] = 4 * grp + r < nvalid ? sv[r] : -INFINITY;
        sv[4 + r] = 16 + 4 * grp + r < nvalid ? sv[4 + r] : -INFINITY;
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])),
                     fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
    mx = wave_max16(mx);
    const float m_new = fmaxf(m, mx);
    const float m_sub = finite_max(m_new);
    const float alpha = fast_exp2(m - m_sub);
    float pv[8];
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      pv[r] = fast_exp2(sv[r] - m_sub);
      ps += pv[r];
    }
    lpart = lpart * alpha + ps;
    m = m_new;
    u32x4 pb;
    pb[0] = pack_bf16x2(pv[0], pv[1]);
    pb[1] = pack_bf16x2(pv[2], pv[3]);
    pb[2] = pack_bf16x2(pv[4], pv[5]);
    pb[3] = pack_bf16x2(pv[6], pv[7]);
    const bf16x8 pfrag = as_bf16x8(pb);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      u32x2 va = f.v[0][db], vb = f.v[1][db];
      if (nvalid < 32) {
        va = mask_v4(va, 4 * grp, nvalid);
        vb = mask_v4(vb, 16 + 4 * grp, nvalid);
      }
      u32x4 vv = {va[0], va[1], vb[0], vb[1]};
      f32x4 c = acc[db];
#pragma unroll
      for (int r = 0; r < 4; ++r) c[r] *= alpha;
      acc[db] = mfma16(as_bf16x8(vv), pfrag, c);
    }
  };

  // two-stage register pipeline: the next step's loads are in flight while this one is
  // multiplied (the load after the last step reads stand-in blocks and is discarded)
  DecodeFrag<D> fa, fb;
  decode_load<D>(fa, k_cache, v_cache, block_off(0), block_off(1), col, grp);
  for (int t0 = k0, sb = 0;; t0 += 64, sb += 4) {
    if (sb == 64) {  // step into the next chunk of the table
      sb = 0;
      ++chunk;
      tab = tab_next;
      tab_next = load_chunk(chunk + 1);
    }
    decode_load<D>(fb, k_cache, v_cache, block_off(sb + 2), block_off(sb + 3), col, grp);
    compute(fa, t0);
    if (t0 + 32 >= k1) break;
    decode_load<D>(fa, k_cache, v_cache, block_off(sb + 4), block_off(sb + 5), col, grp);
    compute(fb, t0 + 32);
    if (t0 + 64 >= k1) break;
  }
#pragma unroll
  for (int db = 0; db < DB; ++db) acc_out[db] = acc[db];
  m_out = m;
  lpart_out = lpart;
}

// The query operand of kv head kvh: lane (col, grp) holds dims 32 kk + 8 grp .. +7 of query
// head kvh * g + col (zeros past the group's heads).
template <int D>
__device__ __forceinline__ void decode_load_q(const uint16_t* __restrict__ q, int i, int hq,
                                              int g, int kvh, bf16x8 (&qf)[D / 32]) {
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (col < g) v = ld16(q + ((size_t)i * hq + kvh * g + col) * D + kk * 32 + grp * 8);
    qf[kk] = as_bf16x8(v);
  }
}

// A decode launch's work list. Work item = (sequence rank, kv head, split); a sequence is cut
// into splits of split_keys keys, and an item's keys into `parts` shares, one per wave
// (parts = 1: one wave is the item). max_keys bounds every length (see decode_cut): a length
// above it breaks the caller's contract and is cut to it (the merge cuts it the same way), so
// such a call computes over fewer keys but never leaves its workspace or the table. A cut
// length's splits all start below it, so no split is empty.
struct DecodeWork {
  const int32_t* seq_lens;
  const int32_t* order;  // sequences longest first, or null: see by_rank
  bool by_rank;          // without an order: each wave ranks the lengths (else: batch order)
  int32_t num_seqs;
  int32_t split_keys, max_splits, max_keys;
};
struct DecodeItem {
  int i, kvh, sp, nsplit, k0, k1;
};
// false: nothing to do (past the list, or past the sequence's splits; 0 splits for a length
// below 1: no output)
__device__ __forceinline__ bool decode_item(const DecodeWork& w, int32_t hkv, int64_t item,
                                            DecodeItem& it) {
  const int64_t per_seq = (int64_t)hkv * w.max_splits;
  const int rank = (int)(item / per_seq);
  if (rank >= w.num_seqs) return false;
  it.i = w.order != nullptr ? w.order[rank]
         : w.by_rank        ? seq_at_rank(w.seq_lens, nullptr, w.num_seqs, rank)
                            : rank;
  const int rem = (int)(item % per_seq);
  it.kvh = rem / w.max_splits;
  it.sp = rem % w.max_splits;
  const int len = min(w.seq_lens[it.i], w.max_keys);
  it.nsplit = (len + w.split_keys - 1) / w.split_keys;
  if (it.sp >= it.nsplit) return false;
  it.k0 = it.sp * w.split_keys;
  it.k1 = min(len, it.k0 + w.split_keys);
  return true;
}

// A work item on one wave.
template <int D>
__device__ __forceinline__ void decode_one_wave(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    int32_t max_blocks, const DecodeWork& work, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale_log2, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    uint16_t* __restrict__ out, float* __restrict__ lse, const DecodeItem& it) {
  constexpr int DB = D / 16;
  const int g = hq / hkv;
  const int lane = threadIdx.x & 63;
  const int col = lane & 15;   // query head within the kv group (column)
  const int grp = lane >> 4;   // lane group 0..3
  const int i = it.i;
  const int h = it.kvh * g + col;
  bf16x8 qf[D / 32];
  decode_load_q<D>(q, i, hq, g, it.kvh, qf);
  f32x4 acc[DB];
  float m, lpart;
  decode_range<D>(qf, k_cache, v_cache, block_tables + (size_t)i * max_blocks, max_blocks, hkv,
                  num_blocks, it.kvh, it.k0, it.k1, scale_log2, acc, m, lpart);
  const float l = wave_sum16(lpart);
  if (col >= g) return;
  if (it.nsplit == 1) {
    const float inv = 1.f / l;
    uint16_t* o = out + ((size_t)i * hq + h) * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      u32x2 w = {pack_bf16x2(acc[db][0] * inv, acc[db][1] * inv),
                 pack_bf16x2(acc[db][2] * inv, acc[db][3] * inv)};
      st8(o + db * 16 + 4 * grp, w);
    }
    if (lse != nullptr && grp == 0) lse[(size_t)i * hq + h] = (m + log2f(l)) * kLn2;
    return;
  }
  const size_t slot = ((size_t)i * hq + h) * work.max_splits + it.sp;
  float* o = ws_o + slot * D;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    f32x4 c = acc[db];
    st16(o + db * 16 + 4 * grp, __builtin_bit_cast(u32x4, c));
  }
  if (grp == 0) {
    ws_ml[slot * 2 + 0] = m;
    ws_ml[slot * 2 + 1] = l;
  }
}

// The body of a one-wave work item.
template <int D>
__device__ __forceinline__ void decode_body(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    int32_t max_blocks, const DecodeWork& work, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale_log2, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    uint16_t* __restrict__ out, float* __restrict__ lse, const int64_t item) {
  DecodeItem it;
  if (!decode_item(work, hkv, item, it)) return;
  decode_one_wave<D>(q, k_cache, v_cache, block_tables, max_blocks, work, hq, hkv, num_blocks,
                     scale_log2, ws_o, ws_ml, out, lse, it);
}

// Keys up to which one wave of a workgroup takes an item alone: with four or eight shares of a
// step or two, the merge and the waves' slots cost more than they save. The host cannot plan for
// it, as it knows the longest length (or a bound above it) only. 256 sequences of 10-100 keys
// under a bound of 4096, 32/8 heads: 23.4 us as four shares, 20.7, 18.2 and 17.8 alone up to 64,
// 96 and 128 keys, 17.3 in a launch of one wave per item; 100 of 60-120, 16/16 heads of 64 dims:
// 14.5, 14.1, 13.0 and 10.6; 4 of 60-120 8.2 each way; 128 of 100-500 under 4096 34.6, 34.6, 34.6
// and 35.1.
constexpr int kLoneKeys = 128;

// Shares' results of one work item on their way to each other.
template <int D, int kParts>
struct DecodeSmem {
  float o[kParts][16][D + 4];  // unnormalised output [share][column][dim] (padded rows)
  float m[kParts][16], l[kParts][16];
};

// The body of a work item run by a workgroup of kWgWaves waves: its keys are cut into kParts
// equal shares (of 32-key steps), wave w takes shares w, w + kWgWaves, ..., and the shares'
// results meet in LDS, where they are merged by their log-sum-exp weights in share order. The
// cut depends on the item's keys only, so the result does not depend on kWgWaves.
template <int D, int kParts, int kWgWaves>
__device__ __forceinline__ void decode_group_body(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    int32_t max_blocks, const DecodeWork& work, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale_log2, float* __restrict__ ws_o, float* __restrict__ ws_ml,
    uint16_t* __restrict__ out, float* __restrict__ lse, const int64_t item,
    DecodeSmem<D, kParts>& sm) {
  static_assert(kParts % kWgWaves == 0, "every wave takes the same number of shares");
  constexpr int DB = D / 16;
  const int g = hq / hkv;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  DecodeItem it;
  if (!decode_item(work, hkv, item, it)) return;  // (workgroup-uniform)
  if (it.k1 - it.k0 <= kLoneKeys) {               // (workgroup-uniform)
    if (wave == 0)
      decode_one_wave<D>(q, k_cache, v_cache, block_tables, max_blocks, work, hq, hkv,
                         num_blocks, scale_log2, ws_o, ws_ml, out, lse, it);
    return;
  }
  const int share = ((it.k1 - it.k0 + kParts - 1) / kParts + 31) / 32 * 32;
  bf16x8 qf[D / 32];
  decode_load_q<D>(q, it.i, hq, g, it.kvh, qf);
#pragma unroll 1
  for (int part = wave; part < kParts; part += kWgWaves) {
    f32x4 acc[DB];
    float m, lpart;
    const int col = lane & 15, grp = lane >> 4;
    const int k0 = it.k0 + part * share;
    if (k0 >= it.k1) {  // an empty share: no weight
      if (lane < 16) sm.m[part][lane] = -INFINITY;
      continue;
    }
    decode_range<D>(qf, k_cache, v_cache, block_tables + (size_t)it.i * max_blocks, max_blocks,
                    hkv, num_blocks, it.kvh, k0, min(it.k1, k0 + share), scale_log2, acc, m,
                    lpart);
    const float l = wave_sum16(lpart);
    if (col < g) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
        st16(&sm.o[part][col][db * 16 + 4 * grp], __builtin_bit_cast(u32x4, acc[db]));
      if (grp == 0) {
        sm.m[part][col] = m;
        sm.l[part][col] = l;
      }
    }
  }
  __syncthreads();
  // one thread per (column, 4 dims), over the shares that have keys
  const int used = (it.k1 - it.k0 + share - 1) / share;
  for (int u = threadIdx.x; u < g * (D / 4); u += 64 * kWgWaves) {
    const int col = u / (D / 4), d = (u % (D / 4)) * 4;
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < kParts; ++s) mx = fmaxf(mx, sm.m[s][col]);
    float den = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kParts; ++s) {
      if (s >= used) break;
      const float w = fast_exp2(sm.m[s][col] - finite_max(mx));
      den += w * sm.l[s][col];
      const f32x4 a = __builtin_bit_cast(f32x4, ld16(&sm.o[s][col][d]));
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] += w * a[e];
    }
    const size_t row = (size_t)it.i * hq + it.kvh * g + col;
    if (it.nsplit == 1) {
      const float inv = 1.f / den;
      st8(out + row * D + d, u32x2{pack_bf16x2(o[0] * inv, o[1] * inv),
                                   pack_bf16x2(o[2] * inv, o[3] * inv)});
      if (lse != nullptr && d == 0) lse[row] = (mx + log2f(den)) * kLn2;
    } else {
      const size_t slot = row * work.max_splits + it.sp;
      st16(ws_o + slot * D + d, __builtin_bit_cast(u32x4, o));
      if (d == 0) {
        ws_ml[slot * 2 + 0] = mx;
        ws_ml[slot * 2 + 1] = den;
      }
    }
  }
}

}  // namespace dec
}  // namespace pkv

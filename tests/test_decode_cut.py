"""CPU tier: how a decode call is cut into work items (csrc/decode_cut.h, host arithmetic alone),
compiled here with the host compiler and swept over the sizes: every split and share that the
kernels form from a sequence's length has keys, lies inside the block table's row, and has a place
in the workspace, also for lengths above the host's max_seq_len."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_23815_amd", "csrc")

SOURCE = """
#include "decode_cut.h"
extern "C" void cut(int32_t num_seqs, int32_t hkv, int32_t max_seq_len, int32_t max_blocks,
                    int64_t* out) {
  const pkv::DecodeCut c = pkv::decode_cut(num_seqs, hkv, max_seq_len, max_blocks);
  out[0] = c.split; out[1] = c.max_splits; out[2] = c.parts; out[3] = c.max_keys;
  out[4] = c.items; out[5] = pkv::decode_split_keys(num_seqs, hkv, max_seq_len);
}
"""


class Cut:
    def __init__(self, v):
        (self.split, self.max_splits, self.parts, self.max_keys, self.items,
         self.base_split) = (int(x) for x in v)


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    gxx = shutil.which("g++") or shutil.which("c++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("cut")
    src, so = d / "cut.cpp", d / "cut.so"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    "-o", str(so), str(src)], check=True)
    fn = ctypes.CDLL(str(so)).cut

    def call(num_seqs, hkv, max_seq_len, max_blocks=None):
        out = (ctypes.c_int64 * 6)()
        fn(num_seqs, hkv, max_seq_len,
           -(-max_seq_len // 16) if max_blocks is None else max_blocks, out)
        return Cut(out)
    return call


def _splits(c, length):
    """The (first key, end) of each split the kernels form for a sequence of this length."""
    n = min(length, c.max_keys)
    return [(s * c.split, min(n, (s + 1) * c.split)) for s in range(-(-n // c.split))]


def _check(c, num_seqs, hkv, max_seq_len, max_blocks):
    what = (num_seqs, hkv, max_seq_len, max_blocks)
    assert c.parts in (1, 4, 8) and c.split % (32 * c.parts) == 0, what
    assert c.items == num_seqs * hkv * c.max_splits, what
    # the workspace is sized for splits of base_split keys
    assert c.max_splits <= -(-max_seq_len // c.base_split), what
    assert c.max_keys >= max_seq_len, what
    rounded = -(-max_seq_len // c.base_split) * c.base_split
    for length in (1, max_seq_len - 1, max_seq_len, max_seq_len + 1, c.max_keys, rounded,
                   rounded + 1, max_blocks * 16, max_blocks * 16 + 5, 2 * max_seq_len):
        if length < 1:
            continue
        splits = _splits(c, length)
        assert len(splits) <= c.max_splits, (what, length)
        # a length above max_seq_len is cut to the workspace's rounding of it and to the table
        assert splits[-1][1] == min(length, rounded, max_blocks * 16), (what, length)
        for k0, k1 in (splits[0], splits[-1]):
            assert 0 <= k0 < k1 <= max_blocks * 16, (what, length, k0, k1)
            share = ((k1 - k0 + c.parts - 1) // c.parts + 31) // 32 * 32
            assert share >= 32 and 1 <= -(-(k1 - k0) // share) <= c.parts, (what, length)


def test_splits_have_keys_inside_the_table(cut):
    rnd = random.Random(0)
    # a last split that would start past the table's row: splits of 4352 keys, lengths rounded
    # to 512 (134912 = 31 x 4352 lies between 8417 x 16 = 134672 and 135168 = 264 x 512)
    c = cut(1, 8, 134672, 8417)
    assert c.split == 4352 and c.base_split == 512
    sizes = [(1, 8, 134672, 8417), (9, 1, 117264, 7329), (1, 8, 300, 19), (256, 8, 4096, 256)]
    for _ in range(20000):
        hkv = rnd.choice([1, 2, 4, 8, 16, 32, 64])
        num_seqs = int(2 ** rnd.uniform(0, 12))
        max_seq_len = int(2 ** rnd.uniform(0, 20))
        blocks = -(-max_seq_len // 16) + rnd.choice([0, 0, 1, 7, 300, 1 << 20])
        sizes.append((num_seqs, hkv, max_seq_len, blocks))
    for s in sizes:
        _check(cut(*s), *s)


def test_split_size_does_not_depend_on_the_table_width(cut):
    """A wider table (rows padded for longer sequences) leaves the cut of the same lengths."""
    rnd = random.Random(1)
    for _ in range(2000):
        num_seqs, hkv = int(2 ** rnd.uniform(0, 10)), rnd.choice([1, 2, 8])
        n = int(2 ** rnd.uniform(0, 18))
        a, b = cut(num_seqs, hkv, n), cut(num_seqs, hkv, n, 1 << 16)
        assert (a.split, a.parts) == (b.split, b.parts)
        assert _splits(a, n) == _splits(b, n)


def test_items_fit_a_grid(cut):
    """Wherever one wave for each split of base_split keys fits a grid of 2^32 - 1 threads, the cut
    does: more pairs and splits than workgroups of several waves have room for go to one wave
    each (129055 x 8 pairs of 17 splits each would be 4.5e9 threads as workgroups of four)."""
    rnd = random.Random(2)
    limit = 2 ** 32 - 1
    sizes = [(129055, 8, 266240), (1 << 17, 8, 1 << 18), (63, 8, 1 << 28), (1 << 20, 1, 600)]
    for _ in range(20000):
        sizes.append((int(2 ** rnd.uniform(0, 24)), rnd.choice([1, 4, 8, 32]),
                      int(2 ** rnd.uniform(0, 28))))
    seen = set()
    for num_seqs, hkv, n in sizes:
        c = cut(num_seqs, hkv, n)
        base_items = num_seqs * hkv * -(-n // c.base_split)
        if base_items * 64 <= limit:
            assert c.items * 64 * c.parts <= limit, (num_seqs, hkv, n, c.parts, c.items)
            seen.add(c.parts)
    assert seen == {1, 4, 8}


def test_short_sequences_of_many_pairs_take_one_wave_each(cut):
    """One wave per item where the pairs fill the chip and the longest sequence has at most a
    third as many keys as there are pairs; four shares past that line, eight for few pairs and
    long sequences."""
    assert [cut(256, 8, n).parts for n in (1, 512, 513, 682, 683, 4096)] == [1, 1, 1, 1, 4, 4]
    assert [cut(384, 8, n).parts for n in (513, 1024, 1025)] == [1, 1, 4]
    assert [cut(512, 8, n).parts for n in (513, 1365, 1366)] == [1, 1, 4]
    assert [cut(255, 8, n).parts for n in (16, 682)] == [4, 4]
    assert [cut(48, 8, n).parts for n in (2047, 2048)] == [4, 8]
    assert [cut(64, 8, n).parts for n in (2047, 2048)] == [4, 4]


def test_long_sequences_of_a_round_and_a_bit_are_split(cut):
    """Eight shares, one item per pair: sequences above 16384 keys are split at 8192, those above
    8192 at 4096 where pairs are few more than compute units; other numbers of pairs and shorter
    sequences keep splits of up to 16384 keys."""
    def n_splits(seqs, n):
        c = cut(seqs, 8, n)
        assert c.parts == 8
        return c.max_splits, min(c.split, 16384)
    for seqs in (17, 32, 33, 40, 41, 63):
        assert n_splits(seqs, 16385) == (3, 8192)
        assert n_splits(seqs, 8192)[0] == 1
    for seqs in (33, 40):
        assert n_splits(seqs, 8193) == (3, 4096)
        assert n_splits(seqs, 16384) == (4, 4096)
    for seqs in (17, 32, 41, 63):
        assert n_splits(seqs, 16384)[0] == 1
    # pairs few enough for two items each: half of 32000 rounded up to 2048 keys
    assert n_splits(16, 32000) == (2, 16384)
    c = cut(64, 8, 32000)
    assert (c.parts, c.split) == (4, 16384)

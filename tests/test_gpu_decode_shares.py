"""GPU tier: the decode plan's cuts (an item's keys shared out among one, four or eight waves of
a workgroup; splits across workgroups) at the sizes where they change, against the fp64 oracle,
and the fused launch's decode half under the same plans, bit for bit."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import bf16_to_f64, dev_pools, say
from tests.test_gpu_decode import check, oracle_decode, run_decode
from tests.test_gpu_mixed import _run, _same

pytestmark = pytest.mark.gpu

CASES = [
    # four shares, one split: shares of one step, of one key, empty last shares
    ("shares4", 8, 2, 128, [0, 1, 31, 32, 33, 95, 96, 127, 128, 129, 1000, 1022, 1023]),
    # four shares, splits of 1024 keys: a last split of one key, of one block
    ("shares4_splits", 4, 1, 64, [1023, 1024, 1039, 1040, 2045]),
    # eight shares, splits of 1024 keys (shares of 128), next to sequences of one split
    ("shares8_splits", 32, 8, 128, [2047, 2048, 3071, 3072, 3073, 40, 1023, 1024]),
    # more than 64 splits of one sequence: the merge takes them in rounds
    ("splits_over_64", 4, 1, 64, [70001, 65, 66000]),
    # 512 pairs and up: four shares, unsplit, longer than 2048 keys
    ("shares4_many", 64, 64, 64, [2100, 5, 300, 2047, 2048, 17, 64, 129]),
    # one wave per item: many pairs of few keys
    ("one_wave", 64, 64, 64, [511, 510, 0, 1, 16, 31, 32, 33] + [7] * 24),
    # the same pairs with one key more
    ("one_wave_edge", 64, 64, 64, [512, 511, 0, 1, 16, 31, 32, 33] + [7] * 24),
    # longest first, the order found by the waves (64 sequences) and by a launch (65)
    ("ranked_64", 32, 32, 128, [600, 0, 5, 5, 17, 599] + [9 + k % 7 for k in range(58)]),
    ("ordered_65", 32, 32, 128, [600, 0, 5, 5, 17, 599] + [9 + k % 7 for k in range(59)]),
    # 2048 pairs: one wave per item up to 682 keys, four shares past them
    ("one_wave_682", 64, 64, 64, [681, 680, 0, 1, 16, 31, 32, 33] + [7] * 24),
    ("shares4_683", 64, 64, 64, [682, 681, 0, 1, 16, 31, 32, 33] + [7] * 24),
    # one wave per item, longest first by a launch (2080 pairs of 128 dims, 420 MB at 412 keys)
    ("one_wave_ordered", 32, 32, 128, [411, 0, 5, 410] + [9 + k % 7 for k in range(61)]),
    # ... and by the waves (32 sequences of 64 pairs each)
    ("one_wave_ranked", 64, 64, 128, [500, 0, 5, 499] + [9 + k % 7 for k in range(28)]),
    # eight shares, few long items (splits of 3584 keys): in the fused launch they come first
    ("shares8_long", 32, 8, 128, [6999, 3583, 3584, 3585, 20, 0] + [50 + k for k in range(10)]),
    # eight shares, 136 pairs above 16384 keys: splits of 8192, a last split of one key
    ("shares8_8192", 8, 8, 64, [16384, 8191, 8192, 16383] + [3 * k for k in range(13)]),
    # 264 pairs above 8192 keys: splits of 4096, a last split of one key
    ("shares8_4096", 8, 8, 64, [8192, 4095, 4096, 8191] + [3 * k for k in range(29)]),
]


def _case(c, prefill=False):
    name, hq, hkv, d, ctx = c
    batches = (W.BatchSpec("decode", len(ctx), W.Dist.const(1), W.Dist.const(1)),)
    if prefill:
        batches = (W.BatchSpec("prefill", 2, W.Dist.const(1), W.Dist.const(1)),) + batches
    spec = W.WorkloadSpec(f"decode_{name}", 180 + CASES.index(c), hq, hkv, d, batches,
                          ("scale", 1.25))
    if prefill:
        return W.make_case(spec, prefix_override=[[40, 300], ctx], new_override=[[70, 9], None])
    return W.make_case(spec, prefix_override=[ctx])


@pytest.mark.parametrize("c", CASES, ids=lambda c: c[0])
def test_decode_shares_match_oracle(gpu_lib, c):
    say(f"[decode shares] {c[0]}")
    case = _case(c)
    check(c[0], run_decode(gpu_lib, case), oracle_decode(case))


@pytest.mark.parametrize("c", CASES, ids=lambda c: c[0])
def test_mixed_decode_shares_equal_the_decode_call(gpu_lib, c):
    say(f"[mixed shares] {c[0]}")
    case = _case(c, prefill=True)
    pk, pv = dev_pools(case)
    sep = _run(gpu_lib, case, False, pools=(pk.clone(), pv.clone()))
    mix = _run(gpu_lib, case, True, pools=(pk, pv))
    assert _same(sep, mix)
    assert all(np.isfinite(x).all() for x in (mix[1], mix[3]))


def test_merge_keeps_an_infinite_value(gpu_lib):
    """An infinite V element under a positive weight makes its output infinite, not NaN, also
    where the merge of the splits reads them in groups that the last one does not fill."""
    say("[decode shares] infinite value")
    name, hq, hkv, d, ctx = CASES[2]
    case = _case(CASES[2])
    b = case.batches[0]
    dim, i = 7, ctx.index(2047)  # two splits of 1024 keys
    case.pool_v[b.block_tables[i, 0], :, dim, 5] = 0x7F80  # +inf at key 5 of every kv head
    out = bf16_to_f64(run_decode(gpu_lib, case)[0])
    assert np.all(np.isposinf(out[i, :, dim]))
    out[i, :, dim] = 0.0
    assert np.isfinite(out).all()


@pytest.mark.parametrize("c", [CASES[1], CASES[2], CASES[3]], ids=lambda c: c[0])
def test_merge_ignores_what_lies_past_the_last_split(gpu_lib, monkeypatch, c):
    """The merge takes eight splits at a time; in a group that the last split does not fill,
    whatever stands in the workspace past its partials stays out of the result (NaN here)."""
    say(f"[decode shares] workspace of NaN, {c[0]}")
    case = _case(c)
    alloc = gpu_lib.alloc_workspace
    monkeypatch.setattr(gpu_lib, "alloc_workspace", lambda n: alloc(n).fill_(0xFF))
    check(c[0], run_decode(gpu_lib, case), oracle_decode(case))

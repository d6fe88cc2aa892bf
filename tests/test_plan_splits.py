"""The planner's automatic splits, on the CPU: every visible pair once (the brute-force check of the
plan tests) on shapes that trigger them, in both dtypes, and a backward workspace that stays within the
psattn_bwd_noalloc array wherever whole ranges and coarse chunks do."""
import pytest

from paper_2608_25683_amd import workloads as W

P = pytest.importorskip("paper_2608_25683_amd.psattn")

from test_abi_host import _check_plan  # noqa: E402

SHAPES = {   # name -> (parent, seg, samples, hq, hkv): what the automatic rules split
    "long_range": ([-1, 0], [700, 20], [1], 8, 2),            # key ranges of few row tiles
    "few_branches": ([-1, 0, 0, 0], [260, 70, 33, 5], [1, 2, 3], 4, 2),
    "one_head": ([-1, 0, 0], [400, 130, 129], [1, 2], 5, 1),
    "short_siblings": ([-1] + [0] * 6, [330, 16, 9, 30, 1, 16, 64], list(range(1, 7)), 8, 2),
}


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_automatic_splits_cover_the_mask(name, dtype):
    parent, seg, samples, hq, hkv = SHAPES[name]
    wl = W.custom(parent, seg, samples, hq=hq, hkv=hkv, dtype=dtype, tensors=False)
    t = P.Tree.from_workload(wl)
    assert t.info["bkv_reduces"] > 0
    _check_plan(wl, t)


def test_automatic_splits_are_equal_pieces():
    wl = W.custom([-1, 0], [4096, 48], [1], hq=4, hkv=4, tensors=False)
    t = P.Tree.from_workload(wl)
    f, m = t.plan_array("fwd_items"), t.plan_array("fwd_merges")
    assert len(m)
    for q_off, nq, part0, nparts in m:
        tiles = (f[(f[:, 0] == q_off) & (f[:, 5] == 0), 3] + 63) // 64
        assert len(tiles) == nparts and tiles.max() - tiles.min() <= nparts


@pytest.mark.parametrize("hq,hkv,prefix,branches,seg", [(28, 4, 3434, 7, 928), (64, 8, 2048, 8, 1800), (40, 8, 1487, 12, 300)])
def test_automatic_splits_stay_within_the_noalloc_array(hq, hkv, prefix, branches, seg):
    wl = W.custom([-1] + [0] * branches, [prefix] + [seg] * branches, list(range(1, branches + 1)), hq=hq, hkv=hkv,
                  tensors=False)
    limit = P.NOALLOC_SCRATCH_MIB << 20
    coarse = P.Tree.from_workload(wl, opts={"fwd_kv_split": -1, "bwd_q_chunk": 1 << 20}).workspace_size(1)
    assert coarse <= limit
    assert P.Tree.from_workload(wl).workspace_size(1) <= limit

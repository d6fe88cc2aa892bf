"""The planner's automatic splits, on the CPU: every visible pair once (the brute-force check of the
plan tests) on shapes that trigger them, in both dtypes, and a backward workspace that stays within the
psattn_bwd_noalloc array wherever whole ranges and coarse chunks do."""
import pytest

from paper_2608_25683_amd import workloads as W

P = pytest.importorskip("paper_2608_25683_amd.psattn")

from test_abi_host import _check_plan, _visible_pairs  # noqa: E402

SHAPES = {   # name -> (parent, seg, samples, hq, hkv): what the automatic rules split
    "long_range": ([-1, 0], [700, 20], [1], 2, 1),            # key ranges of few row tiles
    "long_range_odd": ([-1, 0, 0], [640, 40, 33], [1, 2], 3, 1),
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
    if "long" in name:   # key ranges in pieces, too
        assert len(t.plan_array("merge_launch")) > 0
    _check_plan(wl, t)
    _check_cover(wl, t, dtype == "bf16")


def test_automatic_splits_are_equal_pieces():
    wl = W.custom([-1, 0], [4096, 48], [1], hq=4, hkv=4, tensors=False)
    t = P.Tree.from_workload(wl)
    f, m = t.plan_array("fwd_items"), t.plan_array("fwd_merges")
    assert len(m)
    for q_off, nq, part0, nparts in m:
        tiles = (f[(f[:, 0] == q_off) & (f[:, 5] == 0), 3] + 63) // 64
        assert len(tiles) == nparts and tiles.max() - tiles.min() <= nparts


def test_a_long_range_is_split_among_any_number_of_trees():
    # a cached 300000-token prefix and 16 rows, among more one-token trees than the planner's bound on pieces
    n = 66000
    wl = W.custom([-1, 0] + [-1] * n, [300000, 16] + [1] * n, list(range(1, n + 2)), hq=2, hkv=1, d=64, tensors=False,
                  block_policy=W.blocks_exact)
    call, _ = W.call_subset(wl, list(range(1, n + 2)), [0])
    f = P.Tree.from_workload(call).plan_array("fwd_launch")
    assert f[:, 3].max() <= 32 * 64


def test_long_ranges_are_split_where_fine_pieces_do_not_fit():
    # in pieces of 32 key tiles its partial rows would be more than the psattn_bwd_noalloc array holds
    wl = W.custom([-1, 0], [20000, 16], [1], hq=2, hkv=1, tensors=False)
    t = P.Tree.from_workload(wl)
    assert t.plan_array("fwd_launch")[:, 3].max() <= 10000 and t.workspace_size(1) <= P.NOALLOC_SCRATCH_MIB << 20


def test_chunks_of_consumer_rows_fill_the_compute_units():
    # 47 key tiles whose even share of 256 units is 5 and a bit: 6 equal chunks each would be a second round of
    # a few; longest first over the units, the end is within an eighth of the even share
    wl = W.custom([-1] + [0] * 64, [6000] + [300] * 64, list(range(1, 65)), hq=2, hkv=1, tensors=False)
    rows = sorted((int(n) for n in P.Tree.from_workload(wl).plan_array("bkv_items")[:, 4]), reverse=True)
    units = [0] * 256
    for n in rows:
        units[units.index(min(units))] += n
    assert max(units) <= 1.125 * sum(rows) / 256


@pytest.mark.parametrize("hq,hkv,prefix,branches,seg", [(28, 4, 3434, 7, 928), (64, 8, 2048, 8, 1800), (40, 8, 1487, 12, 300)])
def test_automatic_splits_stay_within_the_noalloc_array(hq, hkv, prefix, branches, seg):
    wl = W.custom([-1] + [0] * branches, [prefix] + [seg] * branches, list(range(1, branches + 1)), hq=hq, hkv=hkv,
                  tensors=False)
    limit = P.NOALLOC_SCRATCH_MIB << 20
    coarse = P.Tree.from_workload(wl, opts={"fwd_kv_split": -1, "bwd_q_chunk": 1 << 20}).workspace_size(1)
    assert coarse <= limit
    assert P.Tree.from_workload(wl).workspace_size(1) <= limit


def _launch_cover(wl, t, bf16, cached=None):
    """(head, row, key row) -> times covered, from the launched items as the kernels read them (cached: slot -> key
    row of keys that are no rows of the call)."""
    G, hc = wl.hq // wl.hkv, t.info["head_chunk"]
    slot_to_row = {**(cached or {}), **({int(s): r for r, s in enumerate(wl.tree.row_slots())})}
    q_list, kv_list, q_pos = t.plan_array("q_list"), t.plan_array("kv_list"), t.plan_array("q_pos")
    cover, written = {}, set()
    for q_off, nq, kv_off, nkv, kv_pos0, head0, part, _ in t.plan_array("fwd_launch"):
        rows, pos = q_list[q_off:q_off + nq], q_pos[q_off:q_off + nq]
        keys = [slot_to_row[int(s)] for s in kv_list[kv_off:kv_off + nkv]]
        if bf16:      # 8 (32-row subtile, head) units of the tile, subtile by subtile
            hk, u0 = head0 // G, head0 % G // hc * 8
            units = [((u0 + i) // G, hk * G + (u0 + i) % G) for i in range(8)]
        else:
            units = [(0, head0)]
        members = [(h, r) for st, h in units for r in range(32 * st, min(nq, 32 * st + 32))]
        assert members, "a launched item without rows"
        for h, r in members:
            if part != -2:
                seen = range(min(nkv, pos[r] - kv_pos0 + 1))
            else:
                pre = nkv - nq
                seen = list(range(pre)) + list(range(pre + r - (pos[r] - pre), pre + r + 1))
            for k in seen:
                x = (h, int(rows[r]), keys[k])
                cover[x] = cover.get(x, 0) + 1
            if part >= 0:
                assert (part + r, h) not in written
                written.add((part + r, h))
    read = {(part0 + j * t.info["q_tile_rows"] + i, h) for _, nq, part0, n in t.plan_array("merge_launch")
            for j in range(n) for i in range(nq) for h in range(wl.hq)}
    assert written == read
    return cover


def _check_cover(wl, t, bf16):
    """The launched items cover every visible pair of a row of the call once per query head, and the launched
    dK/dV items are the listed ones in another order."""
    cover = _launch_cover(wl, t, bf16)
    visible = {(r, k) for r, k in _visible_pairs(wl.tree) if r >= 0}
    assert all(n == 1 for n in cover.values())
    assert {(r, k) for _, r, k in cover} == visible and len(cover) == len(visible) * wl.hq
    listed, launched = (sorted(map(tuple, t.plan_array(a))) for a in ("bkv_items", "bkv_launch"))
    assert listed == launched


@pytest.mark.parametrize("opts", [{}, {"fwd_kv_split": 64}, {"fwd_kv_split": -1}])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (5, 1), (2, 2), (8, 1), (7, 1), (12, 2)])
def test_launched_items_cover_the_mask(hq, hkv, dtype, opts):
    wl = W.custom([-1] + [0] * 7 + [1, 1], [130, 16, 9, 30, 1, 16, 64, 33, 5, 16], list(range(2, 10)), hq=hq, hkv=hkv,
                  dtype=dtype, tensors=False, block_policy=lambda n: W.blocks_fixed(n, 16))
    t = P.Tree.from_workload(wl, opts=opts)
    if opts.get("fwd_kv_split", 0) <= 0:
        assert (t.plan_array("fwd_launch")[:, 6] == -2).any()
    _check_cover(wl, t, dtype == "bf16")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_siblings_under_a_cached_prefix(dtype):
    # packed siblings whose prefix an earlier call computed: as one item, and with the prefix in pieces
    forest = W.custom([-1] + [0] * 6, [330, 16, 9, 14, 1, 12, 16], list(range(1, 7)), hq=8, hkv=2, dtype=dtype, tensors=False)
    call, rows = W.call_subset(forest, list(range(1, 7)), [0])
    for opts, whole in (({"fwd_kv_split": -1}, True), ({"fwd_kv_split": 128}, False)):
        t = P.Tree.from_workload(call, opts=opts)
        assert (t.plan_array("fwd_launch")[:, 6] == -2).any() == whole == (len(t.plan_array("merge_launch")) == 0)
        cover = _launch_cover(call, t, dtype == "bf16", cached={int(s): -1 - i for i, s in enumerate(_cached_slots(forest, 0))})
        # forest rows: the cached node's are its first 330
        want = {(r, k) for r, k in _visible_pairs(forest.tree) if r >= 330}
        got = {(int(rows[r]), -1 - k if k < 0 else int(rows[k])) for _, r, k in cover}
        assert got == want and all(n == 1 for n in cover.values()) and len(cover) == len(want) * forest.hq


def _cached_slots(wl, node):
    tr = wl.tree
    return [s for b in range(tr.blk_ptr[node], tr.blk_ptr[node + 1]) for s in range(tr.blk_base[b], tr.blk_base[b] + tr.blk_len[b])]


@pytest.mark.parametrize("parent,seg,hq,hkv,dtype", [
    ([-1] + [0] * 256, [4096] + [16] * 256, 32, 8, "bf16"), ([-1] + [0] * 1200, [512] + [30] * 1200, 32, 8, "bf16"),
    ([-1] + [0] * 40, [260] + [9] * 40, 10, 2, "bf16"), ([-1] + [0] * 64, [300] + [7] * 64, 4, 2, "fp32")])
def test_unsplit_packs_take_no_workspace(parent, seg, hq, hkv, dtype):
    """Packs of short siblings on whole prefixes write their results directly: no partial rows, no merges, no
    forward workspace, and a backward that holds the row statistics and the dK/dV partial tiles alone."""
    wl = W.custom(parent, seg, list(range(1, len(seg))), hq=hq, hkv=hkv, dtype=dtype, tensors=False)
    t = P.Tree.from_workload(wl, opts={"fwd_kv_split": -1})
    launch = t.plan_array("fwd_launch")
    assert (launch[:, 6] == -2).any() and not (launch[:, 6] >= 0).any()
    assert t.workspace_size(0) == 0 and t.info["fwd_partial_rows"] == 0
    assert t.info["fwd_items"] == len(launch) and t.info["fwd_merges"] == 0 == len(t.plan_array("merge_launch"))
    need = 4 * sum(seg) * hq * 4 + t.info["bkv_partial_tiles"] * 128 * wl.d * 8
    assert t.workspace_size(1) <= need + 8 * 256


@pytest.mark.parametrize("opts", [{}, {"fwd_kv_split": 64}, {"fwd_kv_split": -1}])
@pytest.mark.parametrize("seg", [[512] + [30] * 120, [330, 16, 9, 30, 1, 16, 64], [4096] + [16] * 40])
def test_key_lists_are_no_longer_than_the_paths(seg, opts):
    """Packs share their siblings' lists and add none: what fits the 2^31 entries as paths fits in any plan."""
    wl = W.custom([-1] + [0] * (len(seg) - 1), seg, list(range(1, len(seg))), hq=8, hkv=2, tensors=False)
    t = P.Tree.from_workload(wl, opts=opts)
    assert len(t.plan_array("kv_list")) <= seg[0] + sum(seg[0] + n for n in seg[1:])
    rows = sum(seg)
    assert len(t.plan_array("q_list")) <= 2 * rows + sum(seg[1:])   # tiles; consumers: every node's own and the root's


def test_many_short_branches_fit_the_noalloc_array():
    wl = W.make("c2-small", tensors=False)
    t = P.Tree.from_workload(wl)
    assert t.workspace_size(0) == 0 and t.workspace_size(1) <= P.NOALLOC_SCRATCH_MIB << 20


@pytest.mark.parametrize("opts", [{}, {"fwd_kv_split": 64}, {"fwd_kv_split": -1}])
@pytest.mark.parametrize("name", list(SHAPES))
def test_every_partial_row_is_of_a_launched_tile(name, opts):
    """The workspace holds the launched pieces' rows and nothing else: every tile of q_tile_rows that it has
    belongs to one."""
    parent, seg, samples, hq, hkv = SHAPES[name]
    t = P.Tree.from_workload(W.custom(parent, seg, samples, hq=hq, hkv=hkv, tensors=False), opts=opts)
    bmq, f = t.info["q_tile_rows"], t.plan_array("fwd_launch")
    tiles = {int(p) // bmq for p in f[f[:, 6] >= 0, 6]}
    assert tiles == set(range(t.info["fwd_partial_rows"] // bmq))


@pytest.mark.parametrize("opts", [{}, {"fwd_kv_split": 64}, {"fwd_kv_split": -1}])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (5, 1), (2, 2), (7, 1), (12, 2)])
def test_launched_items_carry_their_limits(hq, hkv, opts):
    """A launched bf16 item's keys end at the last that one of its rows sees, and its unmasked tiles are all those
    that every one of its rows sees whole."""
    wl = W.custom([-1, 0, 0, 1], [300, 161, 33, 90], [2, 3], hq=hq, hkv=hkv, tensors=False)
    t = P.Tree.from_workload(wl, opts=opts)
    G, hc, q_pos = hq // hkv, t.info["head_chunk"], t.plan_array("q_pos")
    for q_off, nq, _, nkv, kv_pos0, head0, part, nfull in t.plan_array("fwd_launch"):
        assert part != -2
        u0 = head0 % G // hc * 8
        rows = [r for i in range(8) for r in range(32 * ((u0 + i) // G), min(nq, 32 * ((u0 + i) // G) + 32))]
        seen = [int(q_pos[q_off + r]) + 1 - kv_pos0 for r in rows]
        assert nkv == max(1, min(nkv, max(seen)))
        assert nfull == max(0, min(nkv, min(seen))) // 64

"""Merging and summing of split results at the edges of the merge kernels: as many pieces as are read
ahead (6), one more, and more pieces than a row's lanes (16 at d = 64, 32 at d = 128).  Against the
fp64 oracle at the bf16 and fp32 tolerances."""
import sys

import pytest

from paper_2608_25683_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import parity_helpers as H  # noqa: E402


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d,keys", [(64, 384), (128, 400), (64, 1030), (128, 2060)])
def test_merge_of_many_pieces(d, keys, dtype):
    # one sequence whose last node's rows see `keys` keys and a few more, in pieces of 64
    wl = W.custom([-1, 0, 0], [keys - 10, 33, 9], [1, 2], hq=2, hkv=1, d=d, dtype=dtype, seed=71)
    print(f"merge d={d} keys={keys} {dtype}", file=sys.stderr, flush=True)
    H.check_full(wl, H.run_gpu(wl, opts={"fwd_kv_split": 64, "bwd_q_chunk": 32}), H.run_oracle(wl))


# 8 (subtile, head) units per forward / dQ item, subtile by subtile, for group sizes that do and do not
# divide 8: rows just below, at and above 32-row subtiles, tiles whose last items have no rows, split
# ranges whose first rows see none of a later piece, and packed siblings
@pytest.mark.parametrize("opts", [None, {"fwd_kv_split": 64, "bwd_q_chunk": 64}])
@pytest.mark.parametrize("hq,hkv,d", [(3, 1, 128), (5, 1, 64), (12, 2, 128), (7, 1, 64), (8, 1, 128), (16, 1, 64)])
def test_items_of_every_group_size(hq, hkv, d, opts):
    wl = W.custom([-1, 0, 0, 1, 0, 0, 0], [161, 33, 130, 64, 7, 12, 1], [2, 3, 4, 5, 6], hq=hq, hkv=hkv, d=d, dtype="bf16",
                  seed=72)
    print(f"units hq={hq} hkv={hkv} d={d} {opts}", file=sys.stderr, flush=True)
    H.check_full(wl, H.run_gpu(wl, opts=opts), H.run_oracle(wl))

"""The fp32 kernels at the edges of their split: 32-row and 32-key tiles dealt out to four
wavefronts, key ranges and row lists that leave some of the wavefronts without work, parts of a
128-key tile past its end, and a cached node whose dK/dV accumulate over two calls.  Against the fp64
oracle at the fp32 tolerance (max-abs and relative L2 1e-5)."""
import sys

import numpy as np
import pytest

from paper_2608_25683_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import parity_helpers as H  # noqa: E402

EDGES = {
    "single_rows": dict(parent=[-1, 0, 0], seg=[1, 2, 1], samples=[1, 2], hq=1, hkv=1, d=128),
    "tile_edges": dict(parent=[-1, 0, 0, 0, 1], seg=[33, 31, 32, 1, 127], samples=[2, 3, 4], hq=4, hkv=2, d=128),
    "key_tile_edges": dict(parent=[-1, 0, 1], seg=[129, 97, 64], samples=[2], hq=3, hkv=1, d=64),
    "many_short": dict(parent=[-1] + [0] * 9, seg=[70] + [5, 16, 1, 16, 9, 33, 2, 15, 17], samples=list(range(1, 10)),
                       hq=5, hkv=1, d=64),
    "long_path": dict(parent=[-1, 0, 1, 1], seg=[300, 260, 40, 7], samples=[2, 3], hq=2, hkv=2, d=128),
}


@pytest.mark.parametrize("opts", [None, {"fwd_kv_split": 64, "bwd_q_chunk": 32}])
@pytest.mark.parametrize("name", list(EDGES))
def test_f32_tile_edges(name, opts):
    c = EDGES[name]
    wl = W.custom(c["parent"], c["seg"], c["samples"], hq=c["hq"], hkv=c["hkv"], d=c["d"], dtype="fp32", sigma=1.0,
                  seed=61, block_policy=lambda n: W.blocks_fixed(n, 24))
    print(f"f32 {name} {opts}", file=sys.stderr, flush=True)
    H.check_full(wl, H.run_gpu(wl, opts=opts), H.run_oracle(wl))


@pytest.mark.parametrize("opts", [None, {"fwd_kv_split": 64, "bwd_q_chunk": 32}])
def test_f32_cached_node_accumulates(opts):
    from paper_2608_25683_amd import psattn as P
    forest = W.custom([-1, 0, 0, 1], [150, 70, 33, 20], [3, 2], hq=4, hkv=2, d=64, dtype="fp32", sigma=1.0, seed=62)
    t = forest.tree
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()
    K, V = up(forest.K_pool), up(forest.V_pool)
    dK, dV = torch.full_like(K, float("nan")), torch.full_like(V, float("nan"))
    out = [np.zeros((t.num_rows, 4, 64)), np.zeros((4, t.num_rows)), np.zeros((t.num_rows, 4, 64))]
    for ends, external in (([3], []), ([2], [0])):
        call, rows = W.call_subset(forest, ends, external)
        tree = P.Tree.from_workload(call, opts=opts, device="cuda")
        print(f"f32 cached call {ends} {opts}", file=sys.stderr, flush=True)
        O, LSE = P.psattn_fwd(tree, up(call.Q), K, V)
        dQ, _, _ = P.psattn_bwd(tree, up(call.Q), K, V, O, LSE, up(call.dO), dK=dK, dV=dV)
        torch.cuda.synchronize()
        out[0][rows], out[1][:, rows], out[2][rows] = O.cpu().numpy(), LSE.cpu().numpy(), dQ.cpu().numpy()
    ref, slots = H.run_oracle(forest), t.row_slots()
    for name, got, want in zip(("O", "LSE", "dQ"), out, ref):
        H.compare(name, got, want, "fp32")
    for name, got, want in (("dK", dK, ref[3]), ("dV", dV, ref[4])):
        H.compare(name, got.double().cpu().numpy()[slots], want[slots], "fp32")

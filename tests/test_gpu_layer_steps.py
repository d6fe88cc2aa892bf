"""The layer steps' kernels at their edges: rotary embedding of ragged row counts, head counts and far
positions."""
import numpy as np
import pytest

from paper_2608_25683_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d,heads,prefix,rows", [(128, 1, 3, 1), (128, 5, 70, 37), (64, 8, 100000, 41), (64, 3, 5, 8)])
def test_rope_against_fp64(d, heads, prefix, rows, dtype, inverse):
    from paper_2608_25683_amd import psattn as P
    wl = W.custom([-1, 0], [prefix, rows], [1], hq=4, hkv=2, d=d, dtype=dtype, tensors=False, block_policy=W.blocks_exact)
    call, _ = W.call_subset(wl, [1], [0])
    tree = P.Tree.from_workload(call, device="cuda")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((rows, heads, d), generator=torch.Generator().manual_seed(5)).to(dt)
    got = P.psattn_rope(tree, x.cuda(), inverse=inverse).double().cpu().numpy()
    pos = np.arange(prefix, prefix + rows, dtype=np.float64)
    ang = (-1 if inverse else 1) * pos[:, None, None] * 10000.0 ** (-np.arange(d // 2) / (d / 2))
    a, b = np.split(x.double().numpy(), 2, axis=-1)
    ref = np.concatenate([a * np.cos(ang) - b * np.sin(ang), a * np.sin(ang) + b * np.cos(ang)], -1)
    # two products and a sum in fp32, sine and cosine rounded to fp32: 4 half-ulps of |a| + |b|; bf16: one
    # more rounding of the result
    size = np.tile(np.abs(a) + np.abs(b), 2)
    bound = 4 * 2.0 ** -24 * size + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0)
    assert np.all(np.abs(got - ref) <= bound + 1e-30)

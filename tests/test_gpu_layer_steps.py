"""The layer steps' kernels at their edges: rotary embedding of ragged row counts, head counts and far
positions, and the bf16 planes of fp32 tensors (exact, any length, special values)."""
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


@pytest.mark.parametrize("n", [1, 3, 4, 1021, 4096, 300000])
def test_planes_hold_the_fp32_value(n):
    from paper_2608_25683_amd import psattn as P
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((n, 1), generator=g, device="cuda") * 10.0 ** torch.randint(-20, 20, (n, 1), generator=g, device="cuda")
    x[0] = torch.finfo(torch.float32).max   # the largest finite value: no plane may overflow
    y = P.psattn_split_planes(x).view(3, n).double()
    assert torch.equal(y.sum(0), x.view(-1).double())
    x = torch.tensor([float("inf"), float("-inf"), float("nan"), 0.0, -0.0], device="cuda").view(-1, 1)
    y = P.psattn_split_planes(x).view(3, -1).float()
    assert torch.equal(torch.nan_to_num(y.sum(0), 7.0), torch.nan_to_num(x.view(-1), 7.0)) and torch.isnan(y[0, 2])


@pytest.mark.parametrize("n,c", [(5, 1), (3, 7), (9, 128)])
def test_silu_bwd_against_fp64(n, c):
    from paper_2608_25683_amd import psattn as P
    g = torch.Generator(device="cuda").manual_seed(c)
    dm = torch.randn((3 * n, c), generator=g, device="cuda")
    a, b = (4 * torch.randn((n, c), generator=g, device="cuda").bfloat16() for _ in range(2))
    da, db = P.psattn_silu_bwd(dm, a, b)
    d, av, bv = dm.view(3, n, c).double().sum(0), a.double(), b.double()
    s = torch.sigmoid(av)
    size = dm.view(3, n, c).double().abs().sum(0)
    # fp32 arithmetic of about ten roundings on terms no larger than size * |b| (1 + |a|)
    for got, ref, top in ((da, d * bv * (s + av * s * (1 - s)), size * bv.abs() * (1 + av.abs())),
                          (db, d * av * s, size * av.abs())):
        assert torch.all((got.view(3, n, c).double().sum(0) - ref).abs() <= 10 * 2.0 ** -24 * top + 1e-30)

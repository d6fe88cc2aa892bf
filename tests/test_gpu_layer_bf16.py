"""The bf16 decoder layer on the GPU: its backward's products run on the bf16 matrix cores with the fp32
gradients as three bf16 planes, and have to hold what fp32 products of the same numbers hold."""
import sys

import numpy as np
import pytest

from paper_2608_25683_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle as O  # noqa: E402

# Gradients from the values that the layer holds: sums of about 3 x 240 exact products in fp32, in an order of the
# library's, and a few fp32 roundings of the operands, 2^-24 each: near 2e-7, at most 1e-6 with every rounding of a
# chain of five steps the same way.  Two planes instead of three leave out the low 8 bits of every element: 9.7e-6 for
# such a product of normal values.
FP32_REL = 1.5e-6
# The whole layer against the exact one: some ten results rounded to bf16 (2^-9) one after the other.
BF16_REL = 10 * 2.0 ** -9


def _mask(s, rows):
    return (np.arange(len(rows)) % 3 != s % 3).astype(float)


@pytest.mark.parametrize("hq,hkv,d,H,F", [(4, 2, 64, 96, 160), (8, 1, 128, 104, 161)])
def test_bf16_layer_backward(hq, hkv, d, H, F, monkeypatch):
    from paper_2608_25683_amd import psattn as P
    from paper_2608_25683_amd.layer import SharedLayer, advantage_adjoint
    wl = W.custom([-1, 0, 0, 1, -1], [90, 40, 25, 33, 51], [3, 2, 4], hq=hq, hkv=hkv, d=d, dtype="bf16", seed=53,
                  block_policy=lambda n: W.blocks_fixed(n, 16), tensors=False)
    t = wl.tree
    ns = t.num_rows
    g = torch.Generator().manual_seed(54)
    draw = lambda shape, s=1.0: (s * torch.randn(shape, generator=g)).bfloat16()
    Wt = {"g1": 1 + draw((H,), 0.1), "Wq": draw((H, hq * d), H ** -0.5), "Wk": draw((H, hkv * d), H ** -0.5),
          "Wv": draw((H, hkv * d), H ** -0.5), "Wo": draw((hq * d, H), (hq * d) ** -0.5), "g2": 1 + draw((H,), 0.1),
          "W1": draw((H, F), H ** -0.5), "W3": draw((H, F), H ** -0.5), "W2": draw((F, H), F ** -0.5)}
    X, c, adv = draw((ns, H)), draw((H,)), np.array([1.5, -0.5, 0.8])
    dout = torch.tensor(advantage_adjoint(t.parent, t.seg_len, t.row_off, t.sample_end, adv, _mask, c.double().numpy()))
    dout += 1e-3 * torch.randn((ns, H), generator=g)         # all 24 bits of a row's gradient in use
    dout = dout.float()
    tree = P.Tree.from_workload(wl, device="cuda")
    layer = SharedLayer({k: v.cuda() for k, v in Wt.items()}, hq, hkv, d)
    Kp = torch.zeros((t.pool_slots, hkv, d), dtype=torch.bfloat16, device="cuda")
    out, s = layer.forward(tree, X.cuda(), Kp, torch.zeros_like(Kp))
    seen = {}
    real_bwd, real_gather = P.psattn_bwd, P.psattn_kv_gather

    def bwd(tree, q, K, V, o, lse, do, **kw):
        seen["do"] = do.clone()
        r = real_bwd(tree, q, K, V, o, lse, do, **kw)
        seen["dq"] = r[0].clone()
        return r

    def gather(*a):
        r = real_gather(*a)
        seen["dk"], seen["dv"] = r[0].clone(), r[1].clone()
        return r
    monkeypatch.setattr(P, "psattn_bwd", bwd)
    monkeypatch.setattr(P, "psattn_kv_gather", gather)
    print(f"bf16 layer hq={hq} hkv={hkv} d={d} H={H} F={F}", file=sys.stderr, flush=True)
    dX, got = layer.backward(tree, s, dout.cuda())
    torch.cuda.synchronize()

    # the same steps in 64 bits, from the activations that the forward saved and from the attention's own results
    f = lambda x: x.detach().double().cpu()
    w = {k: v.double() for k, v in Wt.items()}
    ref, do64 = {}, f(dout)
    ref["W2"] = f(s["m"]).t() @ do64
    dm = do64 @ w["W2"].t()
    a, b = f(s["a"]), f(s["b"])
    sig = torch.sigmoid(a)
    da, db = dm * b * (sig + a * sig * (1 - sig)), dm * a * sig
    ref["W1"], ref["W3"] = f(s["z"]).t() @ da, f(s["z"]).t() @ db
    dz = da @ w["W1"].t() + db @ w["W3"].t()
    yn = f(s["y"]) * f(s["r2"])
    ref["g2"] = (dz * yn).sum(0)
    dzh = dz * w["g2"]
    dy = do64 + (dzh - yn * (dzh * yn).mean(-1, keepdim=True)) * f(s["r2"])
    ref["Wo"] = f(s["o"]).view(ns, hq * d).t() @ dy
    rel = lambda x, y: float((f(x) - y).norm() / y.norm())
    assert rel(seen["do"], (dy @ w["Wo"].t()).view(ns, hq, d)) <= 2.0 ** -8   # rounded to bf16 for the attention
    pos = torch.from_numpy(np.asarray(tree.plan_array("row_pos"), dtype=np.float64))
    ang = -pos[:, None, None] * 10000.0 ** (-torch.arange(d // 2, dtype=torch.float64) / (d / 2))

    def unrotate(x):
        p, q = f(x)[..., :d // 2], f(x)[..., d // 2:]
        return torch.cat([p * torch.cos(ang) - q * torch.sin(ang), p * torch.sin(ang) + q * torch.cos(ang)], -1).reshape(ns, -1)
    dq, dk, dv = unrotate(seen["dq"]), unrotate(seen["dk"]), f(seen["dv"]).reshape(ns, -1)
    h = f(s["h"])
    ref["Wq"], ref["Wk"], ref["Wv"] = h.t() @ dq, h.t() @ dk, h.t() @ dv
    dh = dq @ w["Wq"].t() + dk @ w["Wk"].t() + dv @ w["Wv"].t()
    xn = f(s["X"]) * f(s["r1"])
    ref["g1"] = (dh * xn).sum(0)
    dhh = dh * w["g1"]
    ref["dX"] = dy + (dhh - xn * (dhh * xn).mean(-1, keepdim=True)) * f(s["r1"])
    err = {k: rel(dX if k == "dX" else got[k], v) for k, v in ref.items()}
    print(err, file=sys.stderr, flush=True)
    assert all(e <= FP32_REL for e in err.values()), err


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (8, 1, 128)])
def test_bf16_layer_matches_expanded_samples(hq, hkv, d):
    from paper_2608_25683_amd import psattn as P
    from paper_2608_25683_amd.layer import SharedLayer, advantage_adjoint
    wl = W.custom([-1, 0, 0, 1, -1], [90, 40, 25, 33, 50], [3, 2, 4], hq=hq, hkv=hkv, d=d, dtype="bf16", seed=55,
                  block_policy=lambda n: W.blocks_fixed(n, 16), tensors=False)
    t = wl.tree
    H, F = 96, 160
    g = torch.Generator().manual_seed(56)
    draw = lambda shape, s=1.0: (s * torch.randn(shape, generator=g)).bfloat16()
    Wt = {"g1": 1 + draw((H,), 0.1), "Wq": draw((H, hq * d), H ** -0.5), "Wk": draw((H, hkv * d), H ** -0.5),
          "Wv": draw((H, hkv * d), H ** -0.5), "Wo": draw((hq * d, H), (hq * d) ** -0.5), "g2": 1 + draw((H,), 0.1),
          "W1": draw((H, F), H ** -0.5), "W3": draw((H, F), H ** -0.5), "W2": draw((F, H), F ** -0.5)}
    X, c, adv = draw((t.num_rows, H)), draw((H,)).double().numpy(), np.array([1.5, -0.5, 0.8])
    tree = P.Tree.from_workload(wl, device="cuda")
    layer = SharedLayer({k: v.cuda() for k, v in Wt.items()}, hq, hkv, d)
    Kp = torch.zeros((t.pool_slots, hkv, d), dtype=torch.bfloat16, device="cuda")
    out, s = layer.forward(tree, X.cuda(), Kp, torch.zeros_like(Kp))
    dout = advantage_adjoint(t.parent, t.seg_len, t.row_off, t.sample_end, adv, _mask, c)
    dX, got = layer.backward(tree, s, torch.tensor(dout, dtype=torch.float32, device="cuda"))
    torch.cuda.synchronize()
    ref_out, ref_dX, ref_g = O.layer(t.parent, t.seg_len, t.row_off, t.sample_end, X.double().numpy(),
                                     {k: v.double().numpy() for k, v in Wt.items()}, hq, hkv, wl.scale, 10000.0, 1e-6,
                                     adv, _mask, c)
    for name, x, r in [("out", out, ref_out), ("dX", dX, ref_dX)] + [(k, got[k], ref_g[k]) for k in Wt]:
        rel = float(np.linalg.norm(x.double().cpu().numpy() - r) / np.linalg.norm(r))
        assert rel <= BF16_REL, f"{name}: rel-L2 {rel:.3g} (<= {BF16_REL:.3g})"

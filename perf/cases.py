"""The work that a user of this framework has it do, as cases that can be timed and checked.

Kinds of case:

* ``attn``: prefix-shared attention over one call's forest, through ``psattn_fwd`` (``pass`` "fwd":
  the forward-only pass of log-probabilities) or ``psattn_fwd`` and ``psattn_bwd`` ("step": one
  layer's share of a training step);
* ``rows``: the tree-dependent steps around the attention of a layer: rotary embedding, K/V rows
  into the page pool, dK/dV back into row order, the inverse rotation;
* ``layer``: forward and backward of one whole decoder layer (``SharedLayer``).

Forests are the repository's named workloads (c1 .. c5 and c2-small) or drawn from three
families: ``fan`` (a prompt and its sampled answers), ``chain`` (step-wise trajectories) and
``tree`` (tree sampling).  Structure comes from the case alone; the order of the pool's blocks and
the tensors come from the seed.  Tensors are standard normal, Q, K and V scaled by 0.5 (1.0 for
c1), as in the repository's workloads, so that rows of long prefixes attend over many keys.
"""
import math

import numpy as np
import torch

from paper_2608_25683_amd import psattn as P
from paper_2608_25683_amd import workloads as W
from paper_2608_25683_amd.layer import SharedLayer


def _attn(name, tree, hq=32, hkv=8, d=128, dtype="bf16", what="step", sigma=0.5, **kw):
    return dict(name=name, kind="attn", tree=tree, hq=hq, hkv=hkv, d=d, dtype=dtype, sigma=sigma,
                **{"pass": what}, **kw)


def listed():
    return [
        # the smallest call: a tiny fp32 tree (4 heads, d = 64), the size of a unit test or a smoke
        # run before a job; launches and latency count
        _attn("c1_step_fp32", "c1", 4, 4, 64, "fp32", sigma=1.0),
        # a small bf16 training call: one short prompt and a group of eight short answers, whose
        # buffers are allocated by the call, as the decoder layer does
        _attn("small_step", "fan", prefix=512, branches=8, seg=96, page=16, fresh=True),
        # a micro-batch that continues 16 sequences after cached prefixes (inter-batch sharing):
        # the backward adds to the cached blocks' gradients
        _attn("cached_step", "fan", prefix=1024, branches=16, seg=256, page=64, own=True, cached=True),
        # an fp32 run of step-wise trajectories, as used to check a bf16 run against full precision
        _attn("chains_step_fp32", "chain", 16, 4, 128, "fp32", trees=4, depth=4, lo=64, hi=256, tree_seed=11, page=16),
        # the forward-only pass (reference model, old-policy log-probs) over a 4096-token prompt and
        # 16 answers of 1024
        _attn("c2_fwd", "c2", what="fwd"),
        # the same batch's training step: the headline workload
        _attn("c2_step", "c2"),
        # many tiny branches on a long prompt
        _attn("c2_small_step", "c2-small"),
        # step-wise trajectories of ragged steps, mixed block sizes
        _attn("c3_step", "c3"),
        # tree sampling, branching 4, ragged segments
        _attn("c4_step", "c4"),
        # a forest of 32 trees with log-normal segments, five query heads per kv head: the largest
        _attn("c5_step", "c5", 40, 8, 128),
        # the page-table and rotary steps of a layer over the rows of the tree-sampling batch
        dict(name="c4_rows", kind="rows", tree="c4", hq=32, hkv=8, d=128, dtype="bf16"),
        # a whole decoder layer, forward and backward, with Llama-3-8B's head shape
        dict(name="layer_step", kind="layer", tree="fan", prefix=1024, branches=8, seg=128, page=64, hq=32, hkv=8,
             d=128, hidden=4096, ffn=14336, dtype="bf16"),
    ]


_MAX_FLOPS = {"bf16": 1.4e13, "fp32": 4e10}   # of a drawn attention case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tree(rng, rows_max):
    fam = rng.choice(["fan", "chain", "tree"])
    page = rng.choice([0, 16, 32, 64, 128])       # 0: one block of exactly the segment's length
    if fam == "fan":
        c = dict(tree="fan", prefix=_log_int(rng, 96, 6000), branches=_log_int(rng, 2, 128), seg=_log_int(rng, 8, 1100),
                 page=page)
        if rng.random() < 0.25:
            c.update(own=True, cached=True, branches=_log_int(rng, 2, 24))
    elif fam == "chain":
        lo = _log_int(rng, 16, 400)
        c = dict(tree="chain", trees=_log_int(rng, 1, 12), depth=rng.randint(2, 9), lo=lo, hi=lo * rng.randint(2, 5),
                 tree_seed=rng.randrange(1 << 30), page=page)
    else:
        lo = _log_int(rng, 16, 200)
        c = dict(tree="tree", root=_log_int(rng, 64, 2500), branching=rng.randint(2, 5), depth=rng.randint(1, 3), lo=lo,
                 hi=lo * rng.randint(2, 5), tree_seed=rng.randrange(1 << 30), page=page)
    s = _structure(c)
    return c if sum(s["seg"]) <= rows_max else None


def draw(rng):
    while True:
        kind = rng.choices(["attn", "rows", "layer"], [10, 1, 1])[0]
        if kind == "layer":
            c = _draw_tree(rng, 2200)
            if c is None or c.get("cached"):
                continue
            hq, hkv = rng.choice([(16, 4), (32, 8), (16, 16), (20, 4)])
            h = rng.choice([1024, 2048, 4096])
            c.update(kind="layer", hq=hq, hkv=hkv, d=rng.choice([64, 128]), hidden=h, ffn=h * 7 // 2, dtype="bf16")
            return c
        c = _draw_tree(rng, 60000)
        if c is None:
            continue
        if kind == "rows":
            if c.get("cached"):
                continue
            hq, hkv = rng.choice([(32, 8), (40, 8), (16, 16)])
            c.update(kind="rows", hq=hq, hkv=hkv, d=rng.choice([64, 128]), dtype="bf16")
            return c
        dtype = rng.choices(["bf16", "fp32"], [5, 1])[0]
        hq, hkv = rng.choice([(32, 8), (32, 8), (40, 8), (16, 16), (32, 4), (16, 8), (28, 4)] if dtype == "bf16" else
                             [(4, 4), (16, 4), (8, 2), (10, 2)])
        c.update(kind="attn", hq=hq, hkv=hkv, d=rng.choice([64, 128, 128]), dtype=dtype, sigma=0.5,
                 **{"pass": rng.choices(["step", "fwd"], [3, 1])[0]})
        if 14 * c["d"] * hq * _pairs(_structure(c)) <= _MAX_FLOPS[dtype]:
            return c


# ------------------------------------------------------------------------------ forests

def _structure(case):
    """parent, seg, blocks (per node: (capacity, len)), samples and the cached (external) nodes."""
    name = case["tree"]
    if name in W.CONFIGS:
        t, _ = W.make_tree(name)
        blocks = [[(int(t.blk_cap[b]), int(t.blk_len[b])) for b in range(t.blk_ptr[n], t.blk_ptr[n + 1])]
                  for n in range(t.num_nodes)]
        return dict(parent=[int(x) for x in t.parent], seg=[int(x) for x in t.seg_len], blocks=blocks,
                    samples=[int(x) for x in t.sample_end], external=set())
    external = set()
    if name == "fan" and case.get("own"):          # every answer after a prompt of its own
        n = case["branches"]
        parent = [x for i in range(n) for x in (-1, 2 * i)]
        seg = [case["prefix"], case["seg"]] * n
        samples = list(range(1, 2 * n, 2))
        if case.get("cached"):
            external = set(range(0, 2 * n, 2))
    elif name == "fan":
        parent = [-1] + [0] * case["branches"]
        seg = [case["prefix"]] + [case["seg"]] * case["branches"]
        samples = list(range(1, len(seg)))
    else:
        rng = np.random.default_rng(case["tree_seed"])
        length = lambda: int(rng.integers(case["lo"], case["hi"] + 1))
        parent, seg = [], []
        if name == "chain":
            for _ in range(case["trees"]):
                for k in range(case["depth"]):
                    parent.append(len(seg) - 1 if k else -1)
                    seg.append(length())
            samples = list(range(len(seg)))
        else:
            parent, seg, level = [-1], [case["root"]], [0]
            for _ in range(case["depth"]):
                nxt = []
                for p in level:
                    for _c in range(case["branching"]):
                        parent.append(p)
                        seg.append(length())
                        nxt.append(len(seg) - 1)
                level = nxt
            samples = level
    blocks = [W.blocks_fixed(n, case["page"]) if case["page"] else W.blocks_exact(n) for n in seg]
    return dict(parent=parent, seg=seg, blocks=blocks, samples=samples, external=external)


def _offsets(s):
    off = []
    for p, _n in zip(s["parent"], s["seg"]):
        off.append(0 if p < 0 else off[p] + s["seg"][p])
    return off


def _pairs(s):
    """Visible (query, key) pairs per head."""
    return sum(n * o + n * (n + 1) // 2
               for i, (n, o) in enumerate(zip(s["seg"], _offsets(s))) if i not in s["external"])


def _layout(case, seed):
    """The descriptor's arrays: pool blocks in an order drawn from the seed, rows in node order."""
    s = _structure(case)
    off = _offsets(s)
    blk_ptr, cap, ln, pos = [0], [], [], []
    for i, blocks in enumerate(s["blocks"]):
        at = off[i]
        for c, n in blocks:
            cap.append(c)
            ln.append(n)
            pos.append(at)
            at += n
        blk_ptr.append(len(cap))
    base = np.zeros(len(cap), dtype=np.int64)
    cur = 0
    for b in np.random.default_rng(seed).permutation(len(cap)):
        base[b] = cur
        cur += cap[b]
    row_off, rows = [], 0
    for i, n in enumerate(s["seg"]):
        row_off.append(-1 if i in s["external"] else rows)
        rows += 0 if i in s["external"] else n
    slots = [np.concatenate([np.arange(base[b], base[b] + ln[b]) for b in range(blk_ptr[i], blk_ptr[i + 1])])
             for i in range(len(s["seg"]))]
    return dict(s, off=off, blk_ptr=blk_ptr, cap=cap, len=ln, pos=pos, base=base, pool=int(cur), row_off=row_off, rows=rows,
                slots=slots)


def _tree(case, lay):
    return P.Tree(lay["parent"], lay["seg"], lay["row_off"], lay["blk_ptr"], lay["base"], lay["cap"], lay["len"], lay["pos"],
                  lay["pool"], lay["samples"], case["hq"], case["hkv"], case["d"], 1.0 / math.sqrt(case["d"]),
                  dtype=case["dtype"], device="cuda")


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def __call__(self, shape, dtype, sigma=1.0):
        return (torch.randn(shape, generator=self.g, device="cuda") * sigma).to(dtype)


def _attn_inputs(case, lay, seed):
    draw_, dt = _Draw(seed), _dtype(case)
    q, kv, sg = (lay["rows"], case["hq"], case["d"]), (lay["pool"], case["hkv"], case["d"]), case["sigma"]
    return dict(Q=draw_(q, dt, sg), K=draw_(kv, dt, sg), V=draw_(kv, dt, sg), dO=draw_(q, dt))


def _rows_inputs(case, lay, seed):
    draw_ = _Draw(seed)
    q, kv, n = (lay["rows"], case["hq"], case["d"]), (lay["pool"], case["hkv"], case["d"]), lay["rows"]
    rows = (n, case["hkv"], case["d"])
    return dict(q=draw_(q, _dtype(case)), k=draw_(rows, _dtype(case)), v=draw_(rows, _dtype(case)),
                dq=draw_(q, torch.float32), dK=draw_(kv, torch.float32), dV=draw_(kv, torch.float32))


def _layer_inputs(case, lay, seed):
    draw_, dt = _Draw(seed), _dtype(case)
    h, f, q, kv = case["hidden"], case["ffn"], case["hq"] * case["d"], case["hkv"] * case["d"]
    w = {"g1": 1 + 0.1 * draw_((h,), torch.float32), "g2": 1 + 0.1 * draw_((h,), torch.float32)}
    w = {k: x.to(dt) for k, x in w.items()}
    for k, (a, b) in {"Wq": (h, q), "Wk": (h, kv), "Wv": (h, kv), "Wo": (q, h), "W1": (h, f), "W3": (h, f),
                      "W2": (f, h)}.items():
        w[k] = draw_((a, b), dt, 1.0 / math.sqrt(a))
    return dict(W=w, X=draw_((lay["rows"], h), dt), dout=draw_((lay["rows"], h), torch.float32))


# ------------------------------------------------------------------------------ the calls

def prepare(case, seed):
    lay = _layout(case, seed)
    st = dict(case=case, tree=_tree(case, lay))
    kv = (lay["pool"], case["hkv"], case["d"])
    if case["kind"] == "layer":
        st.update(_layer_inputs(case, lay, seed))
        st["layer"] = SharedLayer(st["W"], case["hq"], case["hkv"], case["d"])
        st["K"] = torch.zeros(kv, dtype=_dtype(case), device="cuda")
        st["V"] = torch.zeros_like(st["K"])
        return st
    if case["kind"] == "rows":
        st.update(_rows_inputs(case, lay, seed))
        # the buffers that a layer's projections and its attention backward write anew each time
        st.update(q_buf=torch.empty_like(st["q"]), k_buf=torch.empty_like(st["k"]), dq_buf=torch.empty_like(st["dq"]))
        st["K"] = torch.zeros(kv, dtype=_dtype(case), device="cuda")
        st["V"] = torch.zeros_like(st["K"])
        return st
    st.update(_attn_inputs(case, lay, seed))
    if not case.get("fresh"):
        st["O"] = torch.empty_like(st["Q"])
        st["LSE"] = torch.empty((case["hq"], lay["rows"]), dtype=torch.float32, device="cuda")
        st["O_lo"] = torch.empty_like(st["Q"]) if case["dtype"] == "bf16" and case["pass"] == "step" else None
        if case["pass"] == "step":
            st["dQ"] = torch.empty(st["Q"].shape, dtype=torch.float32, device="cuda")
            st["dK"] = torch.empty(kv, dtype=torch.float32, device="cuda")
            st["dV"] = torch.empty_like(st["dK"])
    return st


def run(st):
    case, tree = st["case"], st["tree"]
    if case["kind"] == "layer":
        out, saved = st["layer"].forward(tree, st["X"], st["K"], st["V"])
        dx, g = st["layer"].backward(tree, saved, st["dout"])
        return dict(out=out, dX=dx, **{k: g[k] for k in sorted(g)})
    if case["kind"] == "rows":
        q, k, dq = st["q_buf"].copy_(st["q"]), st["k_buf"].copy_(st["k"]), st["dq_buf"].copy_(st["dq"])
        P.psattn_rope(tree, q)
        P.psattn_rope(tree, k)
        P.psattn_kv_scatter(tree, k, st["v"], st["K"], st["V"])
        dk, dv = P.psattn_kv_gather(tree, st["dK"], st["dV"])
        P.psattn_rope(tree, dq, inverse=True)
        P.psattn_rope(tree, dk, inverse=True)
        return dict(q=q, K=st["K"], V=st["V"], dq=dq, dk=dk, dv=dv)
    if case["pass"] == "fwd":
        o, lse = P.psattn_fwd(tree, st["Q"], st["K"], st["V"], st["O"], st["LSE"])
        return dict(O=o, LSE=lse)
    if case.get("fresh"):
        o_lo = torch.empty_like(st["Q"]) if case["dtype"] == "bf16" else None
        o, lse = P.psattn_fwd(tree, st["Q"], st["K"], st["V"], O_lo=o_lo)
        dq, dk, dv = P.psattn_bwd(tree, st["Q"], st["K"], st["V"], o, lse, st["dO"], O_lo=o_lo)
    else:
        if case.get("cached"):      # the accumulators of the cached blocks start a schedule at zero
            st["dK"].zero_()
            st["dV"].zero_()
        o, lse = P.psattn_fwd(tree, st["Q"], st["K"], st["V"], st["O"], st["LSE"], O_lo=st["O_lo"])
        dq, dk, dv = P.psattn_bwd(tree, st["Q"], st["K"], st["V"], o, lse, st["dO"], st["dQ"], st["dK"], st["dV"],
                                  O_lo=st["O_lo"])
    return dict(O=o, LSE=lse, dQ=dq, dK=dk, dV=dv)


# ------------------------------------------------------------------------------ what a pass needs

def work(case):
    s = _structure(case)
    rows = sum(n for i, n in enumerate(s["seg"]) if i not in s["external"])
    pool = sum(c for b in s["blocks"] for c, _n in b)
    keys = sum(s["seg"])
    hq, hkv, d, e = case["hq"], case["hkv"], case["d"], 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "rows":
        # q, k, v rows read and written (k, v into the pool); dq read and written; dK, dV read, dk, dv written
        return {"bytes": rows * d * (2 * hq * e + 4 * hkv * e + 2 * hq * 4 + 4 * hkv * 4), "flops": rows * d * 3 * 2 * (hq + hkv)}
    pairs = _pairs(s)
    if case["kind"] == "layer":
        h, f = case["hidden"], case["ffn"]
        n_w = h * d * (2 * hq + 2 * hkv) + 3 * h * f
        return {"bytes": n_w * (e + 4) + rows * h * (2 * e + 8), "flops": 6 * rows * n_w + 14 * d * hq * pairs}
    q, kv = rows * hq * d, keys * hkv * d
    if case["pass"] == "fwd":
        return {"bytes": 2 * q * e + 2 * kv * e + rows * hq * 4, "flops": 4 * d * hq * pairs}
    return {"bytes": 3 * q * e + q * 4 + 2 * kv * e + 2 * pool * hkv * d * 4 + rows * hq * 4, "flops": 14 * d * hq * pairs}


def tolerance(case):
    # four times the distance between the path and exact(), the largest over a case's outputs
    if case["kind"] == "rows":
        return {"rel": 7e-3}          # seen: 1.7e-3 (bf16 rows), 4e-8 (fp32 rows)
    if case["kind"] == "layer":
        return {"rel": 3.2e-2}        # seen: 7.9e-3 (Wq's gradient)
    # seen: 2.3e-3 (O in bf16); 6e-7 (dK in fp32)
    return {"rel": 9.2e-3} if case["dtype"] == "bf16" else {"rel": 2.4e-6}


# ------------------------------------------------------------------------------ 64-bit results

def _path(lay, n):
    nodes = []
    while n >= 0:
        nodes.append(n)
        n = lay["parent"][n]
    return nodes[::-1]


def _attend(q, k, v, offset, scale):
    """Causal attention of query rows at positions offset .. over keys at 0 ..: q [heads, L, d], one
    kv head's k and v [keys, d].  Returns O, the log-sum-exp and P."""
    s = torch.matmul(q, k.t().contiguous()) * scale
    qpos = offset + torch.arange(q.shape[1], device=q.device)
    s.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > qpos[:, None], -math.inf)
    lse = torch.logsumexp(s, -1)
    p = torch.exp_(s.sub_(lse[..., None]))
    return torch.matmul(p, v), lse, p


def _exact_attn(case, lay, Q, K, V, dO, back):
    """(O, LSE, dQ, dK, dV) in 64 bits, node by node and kv head by kv head."""
    g, scale = case["hq"] // case["hkv"], 1.0 / math.sqrt(case["d"])
    O, dQ = torch.zeros_like(Q), torch.zeros_like(Q)
    LSE = torch.zeros((case["hq"], Q.shape[0]), dtype=torch.float64, device=Q.device)
    dK, dV = torch.zeros_like(K), torch.zeros_like(V)
    for n in range(len(lay["seg"])):
        if n in lay["external"]:
            continue
        slots = torch.from_numpy(np.concatenate([lay["slots"][m] for m in _path(lay, n)])).to(Q.device)
        r = slice(lay["row_off"][n], lay["row_off"][n] + lay["seg"][n])
        for h in range(case["hkv"]):
            hs = slice(h * g, (h + 1) * g)
            q, k, v = Q[r, hs].transpose(0, 1).contiguous(), K[slots, h], V[slots, h]
            o, lse, p = _attend(q, k, v, lay["off"][n], scale)
            O[r, hs], LSE[hs, r] = o.transpose(0, 1), lse
            if not back:
                continue
            do = dO[r, hs].transpose(0, 1).contiguous()
            flat = lambda x: x.reshape(-1, x.shape[-1])
            dV[slots, h] += torch.matmul(flat(p).t().contiguous(), flat(do))
            ds = torch.matmul(do, v.t().contiguous()).sub_((do * o).sum(-1, keepdim=True)).mul_(p).mul_(scale)
            dK[slots, h] += torch.matmul(flat(ds).t().contiguous(), flat(q))
            dQ[r, hs] = torch.matmul(ds, k).transpose(0, 1)
    return O, LSE, dQ, dK, dV


def _rotate(x, pos, theta, sign):
    half = x.shape[-1] // 2
    ang = sign * pos[:, None, None] * theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a, b, c, s = x[..., :half], x[..., half:], torch.cos(ang), torch.sin(ang)
    return torch.cat([a * c - b * s, a * s + b * c], -1)


def _positions(lay):
    pos = [np.arange(o, o + n) for i, (o, n) in enumerate(zip(lay["off"], lay["seg"])) if i not in lay["external"]]
    return torch.from_numpy(np.concatenate(pos)).double().cuda()


def _exact_layer(case, lay, W_, X, dout):
    d, hq, hkv, n = case["d"], case["hq"], case["hkv"], lay["rows"]
    w = {k: v.double() for k, v in W_.items()}
    rms = lambda x: torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + 1e-6)
    mm = lambda a, b: torch.matmul(a, b)
    t = lambda a: a.t().contiguous()
    pos, slot = _positions(lay), torch.from_numpy(np.concatenate(lay["slots"])).cuda()
    r1 = rms(X)
    h = X * r1 * w["g1"]
    q = _rotate(mm(h, w["Wq"]).view(n, hq, d), pos, 10000.0, 1.0)
    k = _rotate(mm(h, w["Wk"]).view(n, hkv, d), pos, 10000.0, 1.0)
    v = mm(h, w["Wv"]).view(n, hkv, d)
    K = torch.zeros((lay["pool"], hkv, d), dtype=torch.float64, device="cuda")
    V = torch.zeros_like(K)
    K[slot], V[slot] = k, v
    o = _exact_attn(case, lay, q, K, V, q, False)[0]
    y = X + mm(o.view(n, -1), w["Wo"])
    r2 = rms(y)
    z = y * r2 * w["g2"]
    a, b = mm(z, w["W1"]), mm(z, w["W3"])
    sig = torch.sigmoid(a)
    m = a * sig * b
    out = y + mm(m, w["W2"])
    g = {"W2": mm(t(m), dout)}
    dm = mm(dout, t(w["W2"]))
    da, db = dm * b * (sig + a * sig * (1 - sig)), dm * a * sig
    g["W1"], g["W3"] = mm(t(z), da), mm(t(z), db)
    dz = mm(da, t(w["W1"])) + mm(db, t(w["W3"]))
    yn = y * r2
    g["g2"] = (dz * yn).sum(0)
    dzh = dz * w["g2"]
    dy = dout + (dzh - yn * (dzh * yn).mean(-1, keepdim=True)) * r2
    g["Wo"] = mm(t(o.view(n, -1)), dy)
    do = mm(dy, t(w["Wo"])).view(n, hq, d)
    _, _, dq, dK, dV = _exact_attn(case, lay, q, K, V, do, True)
    dq = _rotate(dq, pos, 10000.0, -1.0).reshape(n, -1)
    dk = _rotate(dK[slot], pos, 10000.0, -1.0).reshape(n, -1)
    dv = dV[slot].reshape(n, -1)
    g["Wq"], g["Wk"], g["Wv"] = mm(t(h), dq), mm(t(h), dk), mm(t(h), dv)
    dh = mm(dq, t(w["Wq"])) + mm(dk, t(w["Wk"])) + mm(dv, t(w["Wv"]))
    xn = X * r1
    g["g1"] = (dh * xn).sum(0)
    dhh = dh * w["g1"]
    dx = dy + (dhh - xn * (dhh * xn).mean(-1, keepdim=True)) * r1
    return dict(out=out, dX=dx, **{k: g[k] for k in sorted(g)})


def exact(case, seed):
    lay = _layout(case, seed)
    if case["kind"] == "layer":
        x = _layer_inputs(case, lay, seed)
        return _exact_layer(case, lay, x["W"], x["X"].double(), x["dout"].double())
    if case["kind"] == "rows":
        x = {k: v.double() for k, v in _rows_inputs(case, lay, seed).items()}
        pos, slot = _positions(lay), torch.from_numpy(np.concatenate(lay["slots"])).cuda()
        K = torch.zeros((lay["pool"], case["hkv"], case["d"]), dtype=torch.float64, device="cuda")
        V = torch.zeros_like(K)
        K[slot], V[slot] = _rotate(x["k"], pos, 10000.0, 1.0), x["v"]
        return dict(q=_rotate(x["q"], pos, 10000.0, 1.0), K=K, V=V, dq=_rotate(x["dq"], pos, 10000.0, -1.0),
                    dk=_rotate(x["dK"][slot], pos, 10000.0, -1.0), dv=x["dV"][slot])
    x = {k: v.double() for k, v in _attn_inputs(case, lay, seed).items()}
    back = case["pass"] == "step"
    res = dict(zip(("O", "LSE", "dQ", "dK", "dV"), _exact_attn(case, lay, x["Q"], x["K"], x["V"], x["dO"], back)))
    return res if back else dict(O=res["O"], LSE=res["LSE"])

"""The work that users of this library have it do, as measurable cases.

Each case is one pass through the public entry points of ``paper_2609_24802_amd.binding`` on inputs
that already lie on the GPU: fused aggregation over stored CSR graphs (forward, and forward with the
vector-Jacobian product), over the radius, dense and exact kNN relations generated from positions,
the edge-local MLP message, and streaming attention.  ``listed`` names the workloads, ``draw`` gives
more of the same ranges, ``exact`` evaluates a case in 64 bits with plain torch.
"""
import math

import torch

from paper_2609_24802_amd import binding as tb

DEV = "cuda:0"


def listed():
    return [
        # a training step of a small graph layer: one call lasts microseconds, launches and host work count
        dict(name="csr_small_step", op="csr", nodes=1024, edges=8192, feat=16, law="uniform", reducer="sum",
             weighted=True, step=True),
        # inference over a regular graph of degree 32 (a simulation mesh): a tenth of a millisecond
        dict(name="csr_deg32_fwd", op="csr", nodes=131072, edges=131072 * 32, feat=32, law="fixed", reducer="sum",
             weighted=True, step=False),
        # a training step on a power-law graph with hub rows, wide features, reverse incidence kept
        dict(name="csr_powerlaw_step", op="csr", nodes=1_000_000, edges=16_000_000, feat=64, law="powerlaw",
             reducer="sum", weighted=True, step=True),
        # max pooling with its routed gradient; an odd feature width (scalar loads) and ragged sizes
        dict(name="csr_max_f17_step", op="csr", nodes=100_003, edges=1_600_033, feat=17, law="powerlaw",
             reducer="max", weighted=False, step=True),
        # the largest graph: a billion edges resident in HBM, forward
        dict(name="csr_billion_fwd", op="csr", nodes=50_000_000, edges=1_000_000_000, feat=16, law="powerlaw",
             reducer="sum", weighted=True, step=False),
        # a particle model's training step: relation rebuilt from the positions, gradients for both inputs
        dict(name="radius_1m_step", op="radius", n=1_000_000, feat=32, degree=32.0, step=True),
        # a scalar field smoothed over neighbours (density estimate), rebuilt at every call
        dict(name="radius_131k_fwd", op="radius", n=131_072, feat=1, degree=32.0, step=False),
        # direct-sum gravity or electrostatics
        dict(name="dense_65536", op="dense", n=65_536),
        # neighbour sum over the exact kNN relation of a point cloud
        dict(name="knn_131072", op="knn", n=131_072, feat=1, k=16),
        # a long causal prefill
        dict(name="attn_causal_16k", op="attention", n=16_384, heads=16, width=128, dtype="f16", causal=True),
        # bidirectional encoder attention of a ragged length in bfloat16, narrow heads
        dict(name="attn_dense_4001", op="attention", n=4_001, heads=8, width=64, dtype="bf16", causal=False),
        # training step of an edge-local MLP on a scanned surface
        dict(name="edgenn_step", op="edgenn", n=35_947, feat=8, hidden=32, out=3, degree=10.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["csr", "csr", "radius", "radius", "dense", "knn", "attention", "edgenn"])
    if op == "csr":
        feat = rng.choice([1, 3, 8, 16, 17, 32, 50, 64, 128])
        edges = _log(rng, 4_000, min(1 << 25, (1 << 30) // feat))
        nodes = max(64, int(edges / rng.uniform(4, 40)))
        return dict(op=op, nodes=nodes, edges=edges, feat=feat, law=rng.choice(["uniform", "powerlaw"]),
                    reducer=rng.choice(["sum", "sum", "max"]), weighted=rng.random() < 0.7, step=rng.random() < 0.6)
    if op == "radius":
        return dict(op=op, n=_log(rng, 4_000, 1_000_000), feat=rng.choice([1, 4, 8, 15, 16, 31, 32]),
                    degree=round(rng.uniform(8, 32), 2), step=rng.random() < 0.6)
    if op == "dense":
        return dict(op=op, n=_log(rng, 1_000, 65_536))
    if op == "knn":
        return dict(op=op, n=_log(rng, 800, 131_072), feat=rng.choice([1, 3, 4, 8]), k=rng.randint(4, 32))
    if op == "attention":
        return dict(op=op, n=_log(rng, 200, 16_384), heads=rng.randint(1, 16), width=rng.choice([64, 128]),
                    dtype=rng.choice(["f16", "bf16"]), causal=rng.random() < 0.6)
    return dict(op=op, n=_log(rng, 3_000, 60_000), feat=rng.choice([0, 3, 8, 16, 32]),
                hidden=rng.choice([16, 24, 32, 64]), out=rng.randint(1, 8), degree=round(rng.uniform(6, 20), 2))


# ------------------------------------------------------------------------------------- inputs


def _degrees(case, g):
    """In-degrees int64 [nodes] that add up to edges."""
    n, e = case["nodes"], case["edges"]
    if case["law"] == "fixed":
        return torch.full((n,), e // n, dtype=torch.int64, device=DEV)
    if case["law"] == "uniform":
        dst = torch.randint(0, n, (e,), generator=g, device=DEV)
        return torch.bincount(dst, minlength=n)
    # power law of exponent 2.1 (integer part of a Pareto variable), hubs of at most a fiftieth of the edges
    u = torch.rand(n, generator=g, device=DEV).clamp_(min=1e-7)
    cap = float(max(8, min(1_000_000, e // 50)))
    raw = torch.floor(u.pow_(-1.0 / 1.1)).clamp_(max=cap)
    deg = (raw * (e / raw.sum(dtype=torch.float64).item())).clamp_(max=cap).to(torch.int64)
    rest = e - int(deg.sum())
    deg += rest // n
    deg[: rest % n] += 1
    return deg


def _graph(case, g):
    row_ptr = torch.zeros(case["nodes"] + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(_degrees(case, g), 0, out=row_ptr[1:])
    col = torch.randint(0, case["nodes"], (case["edges"],), generator=g, device=DEV, dtype=torch.int32)
    return row_ptr, col


def _cloud(n, degree, g):
    """Points uniform in the unit cube and the radius of the given mean degree."""
    pos = torch.rand(n, 3, generator=g, device=DEV)
    return pos, float(torch.tensor((degree * 3.0 / (4.0 * math.pi * n)) ** (1.0 / 3.0), dtype=torch.float32))


def _surface(n, degree, g):
    """Points on an ellipsoid surface (semi-axes 0.5, 0.45, 0.4) and the radius of the given mean degree."""
    d = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    d /= d.norm(dim=1, keepdim=True)
    pos = (d * torch.tensor([0.5, 0.45, 0.40], dtype=torch.float64, device=DEV)).to(torch.float32)
    area = 4.0 * math.pi * 0.45 ** 2
    return pos, float(torch.tensor(math.sqrt(degree * area / (math.pi * n)), dtype=torch.float32))


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV)
    op = case["op"]
    if op == "csr":
        row_ptr, col = _graph(case, g)
        s = dict(rel=tb.Csr(row_ptr, col, case["nodes"]), x=randn(case["nodes"], case["feat"]), w=None, case=case)
        if case["weighted"]:
            s["w"] = torch.rand(case["edges"], generator=g, device=DEV)
        if case["step"]:
            s["dy"] = randn(case["nodes"], case["feat"])
            s["rev"] = tb.tiga_csr_transpose(s["rel"])
            s["x"].requires_grad_(True)
            if s["w"] is not None:
                s["w"].requires_grad_(True)
        return s
    if op == "radius":
        pos, r = _cloud(case["n"], case["degree"], g)
        s = dict(pos=pos, x=randn(case["n"], case["feat"]), radius=r, sigma=0.5 * r, case=case)
        if case["step"]:
            s["dy"] = randn(case["n"], case["feat"])
            s["pos"].requires_grad_(True)
            s["x"].requires_grad_(True)
        return s
    if op == "dense":
        return dict(pos=randn(case["n"], 3), q=torch.rand(case["n"], generator=g, device=DEV) + 0.5, eps=1e-2, case=case)
    if op == "knn":
        return dict(pos=torch.rand(case["n"], 3, generator=g, device=DEV), x=randn(case["n"], case["feat"]), case=case)
    if op == "attention":
        dt = torch.float16 if case["dtype"] == "f16" else torch.bfloat16
        q, k, v = (randn(case["heads"], case["n"], case["width"]).to(dt) for _ in range(3))
        return dict(q=q, k=k, v=v, case=case)
    pos, r = _surface(case["n"], case["degree"], g)
    F, H, O = case["feat"], case["hidden"], case["out"]
    u = lambda fan, *s: (torch.rand(*s, generator=g, device=DEV) * 2 - 1) / math.sqrt(fan)
    s = dict(pos=pos, x=randn(case["n"], F), radius=r, dy=randn(case["n"], O), W1=u(3 + F, H, 3 + F), b1=u(3 + F, H),
             W2=u(H, O, H), b2=u(H, O), case=case)
    for k in ("pos", "x", "W1", "b1", "W2", "b2"):
        s[k].requires_grad_(True)
    return s


# -------------------------------------------------------------------------------------- passes


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "csr":
        red = tb.REDUCE_MAX if case["reducer"] == "max" else tb.REDUCE_SUM
        if not case["step"]:
            return tb.tiga_mp_csr_fwd(s["rel"], s["x"], s["w"], reducer=red)
        y, arg = tb.csr_aggregate(s["rel"], s["x"], s["w"], reducer=red, rev=s["rev"])
        wrt = (s["x"],) if s["w"] is None else (s["x"], s["w"])
        return (y, arg) + torch.autograd.grad(y, wrt, s["dy"])
    if op == "radius":
        if not case["step"]:
            return tb.tiga_mp_radius_fwd(s["pos"], s["x"], s["radius"], s["sigma"])
        y = tb.radius_aggregate(s["pos"], s["x"], s["radius"], s["sigma"])
        return (y,) + torch.autograd.grad(y, (s["pos"], s["x"]), s["dy"])
    if op == "dense":
        return tb.tiga_mp_dense_fwd(s["pos"], s["q"], s["eps"])
    if op == "knn":
        return tb.tiga_mp_knn_fwd(s["pos"], s["x"], case["k"], want_nbr=True)
    if op == "attention":
        return tb.tiga_mp_attention_fwd(s["q"], s["k"], s["v"], want_lse=True,
                                        relation="triangular" if case["causal"] else "dense")
    y = tb.edge_mlp(s["pos"], s["x"], s["W1"], s["b1"], s["W2"], s["b2"], s["radius"])
    wrt = ("pos", "x", "W1", "b1", "W2", "b2") if case["feat"] else ("pos", "W1", "b1", "W2", "b2")
    return (y,) + torch.autograd.grad(y, [s[k] for k in wrt], s["dy"])


def work(case):
    op = case["op"]
    if op == "csr":
        n, e, f = case["nodes"], case["edges"], case["feat"]
        rows = 4.0 * n * f
        b = 8.0 * (n + 1) + e * (8.0 if case["weighted"] else 4.0) + 2 * rows
        fl = 2.0 * e * f
        if case["reducer"] == "max":
            b += rows
        if case["step"]:  # the reverse incidence, dy and dx; w again and dw; x again (dw) or argmax again
            b += 8.0 * (n + 1) + 4.0 * e + 2 * rows + rows + (8.0 * e if case["weighted"] else 0.0)
            fl += 4.0 * e * f
        return {"bytes": b, "flops": fl}
    if op == "radius":
        n, f, pairs = case["n"], case["feat"], case["n"] * case["degree"]
        b, fl = n * (12.0 + 8.0 * f), pairs * (2.0 * f + 10.0)
        if case["step"]:
            b += n * (24.0 + 12.0 * f)
            fl += pairs * (6.0 * f + 19.0)
        else:
            b += 4.0 * n
        return {"bytes": b, "flops": fl}
    if op == "dense":
        return {"bytes": 28.0 * case["n"], "flops": 20.0 * case["n"] * (case["n"] - 1)}
    if op == "knn":
        n, f, k = case["n"], case["feat"], case["k"]
        # the cells that hold the k nearest and their surroundings: about 8 distances of 8 operations per neighbour
        return {"bytes": n * (12.0 + 8.0 * f + 4.0 * k), "flops": n * k * (64.0 + f)}
    if op == "attention":
        n, h, d = case["n"], case["heads"], case["width"]
        pairs = n * (n + 1) / 2.0 if case["causal"] else float(n) * n
        return {"bytes": h * n * (8.0 * d + 4.0), "flops": 4.0 * d * h * pairs}
    n, f, hd, o = case["n"], case["feat"], case["hidden"], case["out"]
    pairs = n * case["degree"]
    return {"bytes": n * (60.0 + 12.0 * f + 12.0 * o) + 12.0 * hd * (4 + f + o),
            "flops": pairs * 6.0 * hd * (3 + f + o)}


def tolerance(case):
    if case["op"] == "attention":
        # weights and outputs rounded to the input type: unit roundoff 2^-11 or 2^-8
        return {"rel": 1e-3 if case["dtype"] == "f16" else 8e-3, "max": 0.05 if case["dtype"] == "f16" else 0.3}
    if case["op"] == "edgenn":
        # fp32 sums through two layers; a unit within rounding of its threshold may switch
        return {"rel": 2e-6, "max": 1e-2}
    # fp32 sums; neighbour lists, counts and selected edges are decisions of exact fp32 arithmetic
    return {"rel": 1e-6, "max": 1e-4, "differ": 0.0}


# ------------------------------------------------------------------- the same in 64 bits, plain torch


def _pairs(pos, radius):
    """(i, j) of every ordered pair of distinct points whose fp32 squared distance is below fp32(r * r)."""
    n = pos.shape[0]
    p = pos.double()
    lo = p.amin(0)
    h = radius * (1.0 + 1.0 / 1024.0)
    dim = torch.floor((p.amax(0) - lo) / h).long() + 3
    c = torch.floor((p - lo) / h).long() + 1
    key = (c[:, 2] * dim[1] + c[:, 1]) * dim[0] + c[:, 0]
    key, perm = torch.sort(key, stable=True)
    q = pos[perm]
    r2 = torch.tensor(radius, dtype=torch.float32, device=pos.device) ** 2
    got_i, got_j = [], []
    at = torch.arange(n, device=pos.device)
    for dz in (-1, 0, 1):
        for dyy in (-1, 0, 1):
            base = key + (dz * dim[1] + dyy) * dim[0]
            b = torch.searchsorted(key, base - 1)
            e = torch.searchsorted(key, base + 1, right=True)
            for k in range(int((e - b).max())):
                i = at[b + k < e]
                j = b[i] + k
                d = q[j] - q[i]
                d = d * d
                ok = ((d[:, 0] + d[:, 1]) + d[:, 2] < r2) & (i != j)
                got_i.append(perm[i[ok]])
                got_j.append(perm[j[ok]])
    return torch.cat(got_i), torch.cat(got_j)


def _chunks(total, size):
    return [(a, min(total, a + size)) for a in range(0, total, size)]


def _exact_csr(s, case):
    n, e, f = case["nodes"], case["edges"], case["feat"]
    rel, x = s["rel"], s["x"].detach()
    w = None if s["w"] is None else s["w"].detach()
    row_ptr = rel.row_ptr
    y = torch.zeros(n, f, dtype=torch.float64, device=DEV)
    if case["reducer"] == "max":
        if e * f > 1 << 28:
            return None
        row = torch.repeat_interleave(torch.arange(n, device=DEV), row_ptr[1:] - row_ptr[:-1])
        col = rel.col_idx.long()
        m32 = x[col] if w is None else w[:, None] * x[col]
        ix = row[:, None].expand(e, f)
        top = torch.full((n, f), -math.inf, device=DEV).scatter_reduce_(0, ix, m32, "amax")
        eid = torch.arange(e, device=DEV)[:, None].expand(e, f)
        arg = torch.full((n, f), e, device=DEV).scatter_reduce_(
            0, ix, torch.where(m32 == top[row], eid, e), "amin")
        del m32, eid, ix
        ok = arg < e
        a = torch.where(ok, arg, 0)
        src = col[a]
        wv = torch.ones_like(y) if w is None else w.double()[a]
        xv = x.double().gather(0, src)
        y = torch.where(ok, wv * xv, y)
        if not case["step"]:
            return y, None
        dy = torch.where(ok, s["dy"].double(), 0.0)
        dx = torch.zeros_like(y).scatter_add_(0, src, wv * dy)
        if w is None:
            return y, None, dx
        return y, None, dx, torch.zeros(e, dtype=torch.float64, device=DEV).scatter_add_(
            0, a.reshape(-1), (xv * dy).reshape(-1))
    # y: per feature, differences of the running sum over the edges (in 64 bits; rows are consecutive)
    run = torch.zeros(e + 1, dtype=torch.float64, device=DEV)
    for k in range(f):
        m = x[:, k].double().index_select(0, rel.col_idx)
        if w is not None:
            m *= w
        torch.cumsum(m, 0, out=run[1:])
        y[:, k] = run[row_ptr[1:]] - run[row_ptr[:-1]]
    del run, m
    dx = dw = None
    if case["step"]:
        dx = torch.zeros(n, f, dtype=torch.float64, device=DEV)
        dw = None if w is None else torch.zeros(e, dtype=torch.float64, device=DEV)
        for a, b in _chunks(e, max(1, (1 << 29) // f)):
            row = torch.searchsorted(row_ptr, torch.arange(a, b, device=DEV), right=True) - 1
            col = rel.col_idx[a:b].long()
            g = s["dy"].double()[row]
            if w is not None:
                dw[a:b] = (x.double()[col] * g).sum(1)
                g *= w[a:b].double()[:, None]
            dx.index_add_(0, col, g)
    out = (y, None)
    if dx is not None:
        out += (dx,) if dw is None else (dx, dw)
    return out


def _exact_radius(s, case):
    pos, x = s["pos"].detach(), s["x"].detach().double()
    i, j = _pairs(pos, s["radius"])
    p = pos.double()
    sigma = float(torch.tensor(s["sigma"], dtype=torch.float32))
    y = torch.zeros_like(x)
    dx, dpos = torch.zeros_like(x), torch.zeros_like(p)
    for a, b in _chunks(i.numel(), 1 << 22):
        ii, jj = i[a:b], j[a:b]
        d = p[jj] - p[ii]
        k = torch.exp(-(d * d).sum(1) / sigma ** 2)[:, None]
        y.index_add_(0, ii, k * x[jj])
        if case["step"]:
            dy = s["dy"].double()
            dx.index_add_(0, ii, k * dy[jj])
            g = (dy[ii] * x[jj] + dy[jj] * x[ii]).sum(1, keepdim=True)
            dpos.index_add_(0, ii, (2.0 / sigma ** 2) * k * g * d)
    return (y, dpos, dx) if case["step"] else (y, None)


def _exact_dense(s):
    p, q = s["pos"].double(), s["q"].double()
    e2 = float(torch.tensor(s["eps"], dtype=torch.float32) ** 2)
    out = torch.empty_like(p)
    for a, b in _chunks(p.shape[0], 512):
        d = p[None, :, :] - p[a:b, None, :]
        t = q * ((d * d).sum(2) + e2).pow(-1.5)
        out[a:b] = (t[:, :, None] * d).sum(1)
    return out


def _exact_knn(s, case):
    p, x, n, k = s["pos"], s["x"].double(), case["n"], case["k"]
    y = torch.empty_like(x)
    at = torch.arange(n, device=DEV)
    for a, b in _chunks(n, 1024):
        d = p[None, :, :] - p[a:b, None, :]
        d = d * d
        key = (((d[:, :, 0] + d[:, :, 1]) + d[:, :, 2]).view(torch.int32).long() << 32) | at
        key[torch.arange(b - a, device=DEV), at[a:b]] = (1 << 62)
        near = torch.topk(key, k, dim=1, largest=False)[0] & 0xFFFFFFFF
        y[a:b] = x[near].sum(1)
    return y, None


def _exact_attention(s, case):
    H, n, D = s["q"].shape
    y = torch.empty(H, n, D, dtype=torch.float64, device=DEV)
    lse = torch.empty(H, n, dtype=torch.float64, device=DEV)
    scale = float(torch.tensor(D ** -0.5, dtype=torch.float32))
    for h in range(H):
        kt, v = s["k"][h].double().t().contiguous(), s["v"][h].double()
        for a, b in _chunks(n, 4096):
            t = (s["q"][h, a:b].double() @ kt) * scale
            if case["causal"]:
                t.masked_fill_(torch.arange(n, device=DEV)[None, :] > torch.arange(a, b, device=DEV)[:, None], -math.inf)
            lse[h, a:b] = torch.logsumexp(t, 1)
            y[h, a:b] = torch.exp(t - lse[h, a:b, None]) @ v
    return y, lse


def _exact_edgenn(s, case):
    i, j = _pairs(s["pos"].detach(), s["radius"])
    names = ("pos", "x", "W1", "b1", "W2", "b2")
    t = {k: s[k].detach().double().requires_grad_(True) for k in names}
    a = torch.cat([t["pos"][j] - t["pos"][i], t["x"][j]], 1)
    m = torch.relu(a @ t["W1"].t() + t["b1"]) @ t["W2"].t() + t["b2"]
    y = torch.zeros(case["n"], case["out"], dtype=torch.float64, device=DEV).index_add(0, i, m)
    wrt = names if case["feat"] else tuple(k for k in names if k != "x")
    return (y.detach(),) + torch.autograd.grad(y, [t[k] for k in wrt], s["dy"].double())


def exact(case, seed):
    s = prepare(case, seed)
    op = case["op"]
    with torch.enable_grad():
        if op == "csr":
            return _exact_csr(s, case)
        if op == "radius":
            return _exact_radius(s, case)
        if op == "dense":
            return _exact_dense(s)
        if op == "knn":
            return _exact_knn(s, case)
        if op == "attention":
            return _exact_attention(s, case)
        return _exact_edgenn(s, case)

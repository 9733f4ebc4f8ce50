"""The work that programs have this library do, as cases that can be timed and checked.

A case is a dict of plain values.  Its "kind" names the entry points it goes through:

  lp       one LP, from the call until the unscaled answer is there
  batch    many LPs in one block-diagonal solve
  spmv     the plain product with G and with G^T, on device vectors
  project  projections onto rescaled cones, host arrays in and out
  train    one epoch of the warm-start network, then its weights
  predict  a forward pass of the warm-start network

Solves are cut off at ``trials`` trials and, except for conic problems, hold one
restart check (``check``): a solve to a tolerance repeats the same chunk hundreds
of times, but its iterates after the first restart depend on every rounding
before it, so that two correct programs could not be compared there.

``exact`` runs the method (Algorithm 1 up to its first restart, on the rescaled
problem of Section 2.6) and the other cases in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_15504_amd as P


def listed():
    return [
        # the smallest solve: the repository's 200 x 500 problem, every trial bound by latency
        dict(name="lp_small", kind="lp", m=200, n=500, per_col=5, precision="fp64", trials=40, check=40),
        # a member of the warm-start family (2e4 x 4e4, 3e5 nonzeros): an ordinary single LP
        dict(name="lp_mid", kind="lp", m=20000, n=40000, per_col=7.5, precision="fp64", trials=64, check=64),
        # the ill-conditioned problem: row scales 10^U[-3,3], column scales 10^U[-2,2], 5e6 nonzeros
        dict(name="lp_ill", kind="lp", m=200000, n=500000, per_col=10, ill=True, precision="fp64", trials=64, check=64),
        # the large problem's power-law rows (Zipf 1.5, up to 5000 entries) at a quarter of its size
        dict(name="lp_zipf", kind="lp", m=250000, n=500000, zipf=1.5, precision="fp64", trials=64, check=64),
        # the same in mixed precision, kept in single precision by the caller
        dict(name="lp_zipf_mixed", kind="lp", m=250000, n=500000, zipf=1.5, precision="mixed", trials=32, check=32),
        # many small LPs at once
        dict(name="batch_small", kind="batch", count=128, m_lo=60, m_hi=220, cols=2.5, per_col=5, trials=40, check=40),
        # LPs of very different sizes in one batch (m log-uniform from 1e3, n = 2m, 8 per column)
        dict(name="batch_mid", kind="batch", count=48, m_lo=1000, m_hi=20000, cols=2.0, per_col=8, trials=64, check=64),
        # exponential, dual-exponential and second-order-cone rows, up to the first restart check
        dict(name="lp_cones", kind="lp", m_zero=2000, m_nonneg=1000, n_soc=310, n_exp=400, n_dexp=250, n=10000, per_col=3,
             precision="fp64", trials=48, check=64),
        # both products in single precision, as a program with its own outer loop calls them
        dict(name="spmv_zipf", kind="spmv", m=250000, n=500000, zipf=1.5, precision="mixed"),
        # a program's own vectors projected onto diag(f) K_exp
        dict(name="project_exp", kind="project", cone="exp", dim=3, count=131072),
        # an epoch of training on a family of 6000-dimensional members
        dict(name="mlp_train", kind="train", d=6000, width=512, members=8192, batch=256),
        # starts for a batch of members of the 2e4 x 4e4 family
        dict(name="mlp_predict", kind="predict", d=60000, width=512, batch=64),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["lp", "lp", "lp", "batch", "batch", "cones", "spmv", "spmv", "project", "train", "predict"])
    if kind == "lp":
        m = logint(40, 150000)
        per = rng.uniform(3.0, 10.0)
        case = dict(kind="lp", m=m, n=int(m * rng.uniform(1.3, 2.6)), precision=rng.choice(["fp64", "fp64", "mixed"]))
        if m > 20000 and rng.random() < 0.4:
            case["zipf"] = round(rng.uniform(1.45, 1.8), 3)
        else:
            case["per_col"] = round(per, 2)
            case["ill"] = m > 20000 and rng.random() < 0.4
        k = 32 if case["precision"] == "mixed" else 40 if m < 1000 else 64
        return dict(case, trials=k, check=k)
    if kind == "cones":
        q = logint(8, 500)
        return dict(kind="lp", m_zero=logint(20, 3000), m_nonneg=logint(10, 1500), n_soc=int(q * rng.random()),
                    n_exp=int(q * rng.random()), n_dexp=1 + int(q * rng.random()), n=logint(2000, 14000), per_col=3,
                    precision="fp64", trials=rng.randint(32, 56), check=64)
    if kind == "batch":
        if rng.random() < 0.5:
            return dict(kind="batch", count=logint(8, 160), m_lo=rng.randint(30, 80), m_hi=rng.randint(100, 240),
                        cols=round(rng.uniform(1.5, 2.7), 2), per_col=5, trials=40, check=40)
        return dict(kind="batch", count=logint(5, 40), m_lo=logint(600, 2000), m_hi=logint(4000, 22000),
                    cols=round(rng.uniform(1.4, 2.4), 2), per_col=rng.randint(4, 10), trials=64, check=64)
    if kind == "spmv":
        m = logint(300, 220000)
        case = dict(kind="spmv", m=m, n=int(m * rng.uniform(0.7, 2.4)), precision=rng.choice(["fp64", "mixed"]))
        if rng.random() < 0.5:
            return dict(case, zipf=round(rng.uniform(1.45, 1.9), 3))
        return dict(case, per_col=round(rng.uniform(3.0, 11.0), 2))
    if kind == "project":
        cone = rng.choice(["soc", "exp", "exp_dual"])
        dim = 3 if cone != "soc" else logint(2, 300)
        return dict(kind="project", cone=cone, dim=dim, count=logint(64, 390000 // dim))
    if kind == "train":
        return dict(kind="train", d=logint(300, 6000), width=rng.choice([64, 128, 200, 256, 512]),
                    members=logint(300, 6000), batch=rng.choice([64, 100, 128, 256]))
    return dict(kind="predict", d=logint(450, 60000), width=rng.choice([64, 200, 256, 512]), batch=logint(1, 500))


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + salt)


def _lp_data(case, seed):
    """min c^T x, G x - h in the row cones, 0 <= x <= 10: the planted recipe of the repository's
    generators (values N(0,1), h = G x0 - s with s inside the row's cone, c ~ U[0,1])."""
    g, dev = _gen(seed), "cuda"
    soc = [3] * case.get("n_soc", 0)
    soc[::6] = [9] * len(soc[::6])
    soc[::31] = [50] * len(soc[::31])
    ne, nd = case.get("n_exp", 0), case.get("n_dexp", 0)
    cone_rows = sum(soc) + 3 * (ne + nd)
    if "m" in case:
        m, m_zero, m_nonneg = case["m"], case["m"], 0
    else:
        m_zero, m_nonneg = case["m_zero"], case["m_nonneg"]
        m = m_zero + m_nonneg + cone_rows
    n = case["n"]
    if case.get("zipf"):
        cdf = (torch.arange(1, 5001, device=dev, dtype=torch.float64) ** -case["zipf"]).cumsum(0)
        u = torch.rand(m, generator=g, device=dev, dtype=torch.float64) * cdf[-1]
        lengths = (torch.searchsorted(cdf, u) + 1).clamp(max=min(5000, n))
        row = torch.repeat_interleave(torch.arange(m, device=dev), lengths)
        col = torch.randint(n, row.shape, generator=g, device=dev)
    else:
        k = case["per_col"]  # 7.5: eight entries in one half of the columns, seven in the other
        lengths = torch.full((n,), int(k), device=dev)
        lengths[: int(round((k - int(k)) * n))] += 1
        lengths = lengths[torch.randperm(n, generator=g, device=dev)]
        col = torch.repeat_interleave(torch.arange(n, device=dev), lengths)
        row = torch.randint(m, col.shape, generator=g, device=dev)
    key = torch.unique(row * n + col)
    row, col = key // n, key % n
    val = torch.randn(key.shape, generator=g, device=dev, dtype=torch.float64)

    def uniform(count, lo, hi):
        return lo + (hi - lo) * torch.rand(count, generator=g, device=dev, dtype=torch.float64)

    if case.get("ill"):
        val = val * (10.0 ** uniform(m, -3, 3))[row] * (10.0 ** uniform(n, -2, 2))[col]
    x0, c = uniform(n, 0, 5), uniform(n, 0, 1)
    s = torch.zeros(m, device=dev, dtype=torch.float64)
    r = m_zero
    s[r:r + m_nonneg] = uniform(m_nonneg, 0.5, 1.5)
    r += m_nonneg
    for d in soc:
        w = torch.randn(d - 1, generator=g, device=dev, dtype=torch.float64)
        s[r], s[r + 1:r + d] = w.norm() + 1.2, w
        r += d
    a, b, q = uniform(ne, -2, 1), uniform(ne, 0.5, 2), uniform(ne, 1.5, 2.5)
    s[r:r + 3 * ne] = torch.stack([a, b, q * b * torch.exp(a / b)], 1).reshape(-1)
    r += 3 * ne
    a, b, q = uniform(nd, 0.5, 2), uniform(nd, -1, 2), uniform(nd, 1.5, 2.5)
    s[r:] = torch.stack([-a, b, q * a * torch.exp(-b / a - 1)], 1).reshape(-1) if nd else s[r:]
    row, col, val, x0, c, s = (t.cpu().numpy() for t in (row, col, val, x0, c, s))
    h = np.bincount(row, weights=val * x0[col], minlength=m) - s
    ptr = np.zeros(m + 1, np.int64)
    np.cumsum(np.bincount(row, minlength=m), out=ptr[1:])
    return dict(m=m, n=n, m_zero=m_zero, soc=soc, n_exp=ne, n_dexp=nd, row=row, ptr=ptr, col=col.astype(np.int32), val=val,
                h=h, c=c, l=np.zeros(n), u=np.full(n, 10.0))


def _problem(d):
    return P.Problem(d["m"], d["n"], d["m_zero"], d["ptr"], d["col"], d["val"], d["h"], d["c"], d["l"], d["u"], d["soc"],
                     d["n_exp"], d["n_dexp"])


def _members(case):
    """The sizes of a batch: log-uniform between its bounds, without chance."""
    k = case["count"]
    at = [(0.5 + (7 * i) % k) / k for i in range(k)]
    ms = [int(case["m_lo"] * (case["m_hi"] / case["m_lo"]) ** t) for t in at]
    return [dict(m=m, n=int(m * case["cols"]), per_col=min(case["per_col"], m)) for m in ms]


def _vectors(case, seed):
    """Points and factors of the projections: about the size of a solver's residuals, mild row scales."""
    r = np.random.default_rng([int(seed), case["count"], case["dim"]])
    v = 2.0 * r.standard_normal((case["count"], case["dim"]))
    return v, np.exp(r.uniform(-1.2, 1.2, v.shape))


def _net_data(case, seed):
    d, w, g = case["d"], case["width"], _gen(seed)

    def layer(out, inp):
        a = math.sqrt(6.0 / (out + inp))
        return (2 * torch.rand(out, inp, generator=g, device="cuda") - 1) * a

    ws = [layer(w, d), layer(w, w), layer(d, w)]
    bs = [0.01 * torch.randn(k, generator=g, device="cuda") for k in (w, w, d)]
    norm = [torch.randn(d, generator=g, device="cuda"), 0.5 + torch.rand(d, generator=g, device="cuda"),
            torch.randn(d, generator=g, device="cuda"), 0.5 + torch.rand(d, generator=g, device="cuda")]
    rows = case.get("members", case["batch"])
    u = norm[0] + norm[1] * torch.randn(rows, d, generator=g, device="cuda")
    t = norm[2] + norm[3] * torch.randn(rows, d, generator=g, device="cuda") if case["kind"] == "train" else None
    return ws, bs, norm, u, t


def prepare(case, seed):
    if case["kind"] == "lp":
        return dict(case=case, problem=_problem(_lp_data(case, seed)))
    if case["kind"] == "batch":
        problems = [_problem(_lp_data(c, seed * 997 + i)) for i, c in enumerate(_members(case))]
        return dict(case=case, batch=P.Batch(problems))
    if case["kind"] == "spmv":
        d = _lp_data(case, seed)
        t = torch.float64 if case["precision"] == "fp64" else torch.float32
        g = _gen(seed, 1)
        return dict(case=case, problem=_problem(d), x=torch.randn(d["n"], generator=g, device="cuda", dtype=t),
                    y=torch.randn(d["m"], generator=g, device="cuda", dtype=t))
    if case["kind"] == "project":
        v, f = _vectors(case, seed)
        return dict(case=case, v=v, f=f)
    ws, bs, norm, u, t = _net_data(case, seed)
    net = P.MLP(case["d"], case["width"], case["d"])
    net.params = torch.cat([p.reshape(-1) for pair in zip(ws, bs) for p in pair]).cpu().numpy()
    net.set_normalization(*(q.cpu().numpy() for q in norm))
    return dict(case=case, net=net, u=u, t=t)


# ---- one pass ---------------------------------------------------------------------------------------------------------
def _limits(case):
    return dict(max_iter=case["trials"], check_every=case["check"])


def run(state):
    case = state["case"]
    if case["kind"] == "lp":
        big = case["n"] > 50000  # a large answer stays on the device
        s = state["problem"].solve(precision=case["precision"], device_out=big, **_limits(case))
        x, y, lam = s.x, s.y, s.lam
        if case["precision"] == "mixed":
            x, y, lam = (v.float() if big else v.astype(np.float32) for v in (x, y, lam))
        i = s.info
        return dict(x=x, y=y, lam=lam, trials=i["iters"], accepted=i["accepted_iters"], restarts=i["restarts"], omega=i["omega"],
                    pobj=i["pobj"])
    if case["kind"] == "batch":
        sols = state["batch"].solve(device_out=True, precision="fp64", **_limits(case))
        return dict(x=torch.cat([s.x for s in sols]), y=torch.cat([s.y for s in sols]), lam=torch.cat([s.lam for s in sols]),
                    accepted=np.array([s.info["accepted_iters"] for s in sols]), restarts=np.array([s.info["restarts"] for s in sols]))
    if case["kind"] == "spmv":
        x, y = state["x"], state["y"]
        gx, gty = torch.empty_like(y), torch.empty_like(x)
        st = torch.cuda.current_stream().cuda_stream
        state["problem"].spmv(x.data_ptr(), gx.data_ptr(), precision=case["precision"], stream=st)
        state["problem"].spmv(y.data_ptr(), gty.data_ptr(), transpose=True, precision=case["precision"], stream=st)
        return dict(gx=gx, gty=gty)
    if case["kind"] == "project":
        return P.pdcs_project_cone(case["cone"], state["v"], state["f"])
    if case["kind"] == "train":
        u, t, b = state["u"], state["t"], case["batch"]
        losses = [state["net"].train_step(u[lo:lo + b], t[lo:lo + b], 1e-3) for lo in range(0, len(u), b)]
        return dict(losses=np.array(losses), params=state["net"].params)
    return state["net"].forward(state["u"])


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def _nnz(case):
    if not case.get("zipf"):
        return case["n"] * case["per_col"]
    k = np.arange(1, 5001, dtype=np.float64)
    p = k ** -case["zipf"]
    return case["m"] * float((k * p).sum() / p.sum())


def _lp_work(case):
    """Each trial depends on the one before it and reads G by rows and by columns once, its vectors once."""
    n, nnz = case["n"], _nnz(case)
    m = case.get("m") or case["m_zero"] + case["m_nonneg"] + 5 * case["n_soc"] + 3 * (case["n_exp"] + case["n_dexp"])
    s = 8 if case.get("precision") != "mixed" else 4
    trial = 2 * nnz * (s + 4) + s * (19 * n + 10 * m)
    scaling = 2 * nnz * (8 + 4) + 2 * nnz * s
    return trial * case["trials"] + scaling, (4 * nnz + 12 * (n + m)) * case["trials"]


def work(case):
    if case["kind"] == "lp":
        by, fl = _lp_work(case)
    elif case["kind"] == "batch":
        by, fl = map(sum, zip(*(_lp_work(dict(c, trials=case["trials"])) for c in _members(case))))
    elif case["kind"] == "spmv":
        s, nnz = (8 if case["precision"] == "fp64" else 4), _nnz(case)
        by, fl = 2 * nnz * (s + 4) + 2 * s * (case["m"] + case["n"]) + 4 * (case["m"] + case["n"]), 4 * nnz
    elif case["kind"] == "project":
        by, fl = 24 * case["count"] * case["dim"], 40 * case["count"] * case["dim"]
    else:
        d, w, b = case["d"], case["width"], case["batch"]
        weights = 2 * d * w + w * w
        if case["kind"] == "train":
            steps = -(-case["members"] // b)
            by = steps * 26 * weights + 8 * d * case["members"] + 4 * weights
            fl = (6 * weights - 2 * d * w) * case["members"]
        else:
            by, fl = 2 * weights + 8 * d * b, 2 * weights * b
    return dict(bytes=by, flops=fl)


# ---- the same in 64 bits, with plain torch ----------------------------------------------------------------------------
def _exp_projection(v, f):
    """Rows of v onto diag(f) K_exp, K_exp = closure {y > 0, y e^(x/y) <= z}: v inside; 0 in the polar cone; else
    p = s F (r, 1, e^r) with v - p = -t F^-1 (-1, r - 1, e^-r) and s, t > 0, which only the projection meets, or the
    clip onto the face y = 0."""
    out = torch.stack([v[:, 0].clamp(max=0), torch.zeros_like(v[:, 1]), v[:, 2].clamp(min=0)], 1)

    def parts(r, v, f):
        e, ei = torch.exp(r.clamp(max=0)), torch.exp((-r).clamp(max=0))  # e^r and e^-r, each over max(1, e^r), max(1, e^-r)
        up = torch.exp((-r).clamp(max=0))
        a = torch.stack([f[..., 0] * r * up, f[..., 1] * up, f[..., 2] * e], -1)
        k = torch.stack([-e / f[..., 0], e * (r - 1) / f[..., 1], ei / f[..., 2]], -1)
        return a, k, (v * torch.linalg.cross(a, k)).sum(-1)

    # r from -4e8 (rays that have met the face's edge) to 300: steps of 0.015 near 0, of 1.5 percent further out
    grid = torch.sinh(torch.linspace(-20.5, 6.39, 1793, device=v.device, dtype=torch.float64))
    for i in range(0, len(v), 8192):
        w, q = v[i:i + 8192], f[i:i + 8192]
        turn = parts(grid[None, :], w[:, None, :], q[:, None, :])[2]
        at, cell = torch.nonzero((turn[:, :-1] > 0) & (turn[:, 1:] <= 0), as_tuple=True)
        lo, hi, w, q = grid[cell], grid[cell + 1], w[at], q[at]
        for _ in range(80):
            mid = 0.5 * (lo + hi)
            up = parts(mid, w, q)[2] > 0
            lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
        a, k, _ = parts(0.5 * (lo + hi), w, q)
        s = (a * w).sum(-1) / (a * a).sum(-1)
        good = (s > 0) & ((k * w).sum(-1) < 0)
        out[i + at[good]] = (s[:, None] * a)[good]
    x, y, z = (v / f).unbind(1)
    inside = (y > 0) & (z > 0) & (x <= y * torch.log((z / y).clamp(min=1e-300)))
    x, y, z = (-f * v).unbind(1)
    polar = (x < 0) & (z > 0) & (torch.log((-x).clamp(min=1e-300)) + y / x <= 1 + torch.log(z.clamp(min=1e-300)))
    return torch.where(inside[:, None], v, torch.where(polar[:, None], torch.zeros_like(v), out))


def _soc_projection(v, f):
    """Rows of v onto diag(f) {||w|| <= t}: v inside, 0 in the polar cone, else the multiplier by bisection."""
    v0, w, e0, e = v[:, :1], v[:, 1:], f[:, :1], f[:, 1:]
    inside = (w / e).norm(dim=1, keepdim=True) <= v0 / e0
    far = (w * e).norm(dim=1, keepdim=True)
    lo, hi = (-v0 * e0).clamp(min=0), torch.maximum(far, (-v0 * e0).clamp(min=0))
    for _ in range(100):
        mu = 0.5 * (lo + hi)
        s = v0 / e0 + mu / e0 ** 2
        over = ((w * e / (e * e * s + mu)) ** 2).sum(1, keepdim=True) > 1
        lo, hi = torch.where(over, mu, lo), torch.where(over, hi, mu)
    mu = 0.5 * (lo + hi)
    s = v0 / e0 + mu / e0 ** 2
    p = torch.cat([e0 * s, w * e * e * s / (e * e * s + mu)], 1)
    return torch.where(inside, v, torch.where(far <= -v0 * e0, torch.zeros_like(v), p))


def _cone_projection(cone, v, f):
    if cone == "soc":
        return _soc_projection(v, f)
    return _exp_projection(v, f) if cone == "exp" else v + _exp_projection(-v, 1 / f)


def _lp_exact(case, seed):
    d = _lp_data(case, seed)
    m, n = d["m"], d["n"]
    row, col, val, h, c, lo, up = (torch.as_tensor(np.asarray(d[k]), device="cuda") for k in ("row", "col", "val", "h", "c", "l", "u"))
    col = col.long()

    def over(at, size, what, how):
        return torch.zeros(size, device="cuda", dtype=torch.float64).scatter_reduce_(0, at, what, how)

    D1, D2 = torch.ones_like(h), torch.ones_like(c)
    for k in range(11):  # ten Ruiz passes, one pass of square roots of 2-norms
        a = (D1[row] * val) * D2[col]
        how = ("amax", a.abs()) if k < 10 else ("sum", a * a)
        sr, sc = over(row, m, how[1], how[0]), over(col, n, how[1], how[0])
        for D, s in ((D1, sr), (D2, sc)):
            q = s.sqrt() if k < 10 else s.sqrt().sqrt()
            D.copy_(torch.where(s > 0, D / q, D))
    a = (D1[row] * val) * D2[col]
    h, c, lo, up = D1 * h, D2 * c, lo / D2, up / D2
    G = lambda x: over(row, m, a * x[col], "sum")  # noqa: E731
    Gt = lambda y: over(col, n, a * y[row], "sum")  # noqa: E731
    blocks, r = [], d["m_zero"] + (m - d["m_zero"] - sum(d["soc"]) - 3 * (d["n_exp"] + d["n_dexp"]))
    first_cone = r
    soc = {}
    for q in d["soc"]:
        soc.setdefault(q, []).append(r)
        r += q
    for q, starts in soc.items():
        blocks.append(("soc", "soc", torch.tensor(starts, device="cuda")[:, None] + torch.arange(q, device="cuda")))
    for kinds, count in ((("exp", "exp_dual"), d["n_exp"]), (("exp_dual", "exp"), d["n_dexp"])):
        if count:
            blocks.append((*kinds, r + torch.arange(3 * count, device="cuda").reshape(-1, 3)))
        r += 3 * count

    def onto(v, dual):  # K_d of y (dual), K_d* of G x - h
        z = v.clone()
        z[d["m_zero"]:first_cone] = v[d["m_zero"]:first_cone].clamp(min=0)
        if not dual:
            z[: d["m_zero"]] = 0
        for primal_kind, dual_kind, at in blocks:
            z[at] = _cone_projection(dual_kind if dual else primal_kind, v[at], 1 / D1[at] if dual else D1[at])
        return z

    eta, omega = float(1 / a.abs().max()), float(c.norm() / h.norm())
    x = torch.zeros_like(c).clamp(lo, up)
    y = onto(torch.zeros_like(h), True)
    gx, gty = G(x), Gt(y)
    xa, ya, gxa, gtya = x, y, gx, gty
    k = 0
    for trial in range(1, case["trials"] + 1):
        xh = (x - (eta / omega) * (c - gty)).clamp(lo, up)
        gxh = G(xh)
        yh = onto(y + eta * omega * (h - 2 * gxh + gx), True)
        dx, dy = xh - x, yh - y
        num, den = 0.5 * float(omega * dx @ dx + dy @ dy / omega), abs(float(dy @ (gxh - gx)))
        bar = num / den if den > 0 else math.inf
        kept = eta < bar
        eta = min((1 - (trial + 1.0) ** -0.3) * bar, (1 + (trial + 1.0) ** -0.6) * eta)
        gtyh = Gt(yh)
        if not kept:
            continue
        lam = c - gtyh
        res = gxh - h
        pobj, dobj = float(c @ xh), float(h @ yh + lo @ lam.clamp(min=0) - up @ (-lam).clamp(min=0))
        worst = max(float((res - onto(res, False)).norm()) / (1 + float(h.abs().sum())),
                    abs(pobj - dobj) / (1 + abs(pobj) + abs(dobj)))
        beta = min(max(-0.1 * math.log10(worst) + 0.2, 0.0), 1.0) if worst > 0 else 1.0
        w, v = (k + 1.0) / (k + 2.0), 1.0 / (k + 2.0)
        x, y = w * ((1 + beta) * xh - beta * x) + v * xa, w * ((1 + beta) * yh - beta * y) + v * ya
        gx, gty = w * ((1 + beta) * gxh - beta * gx) + v * gxa, w * ((1 + beta) * gtyh - beta * gty) + v * gtya
        k += 1
    return dict(x=D2 * xh, y=D1 * yh, lam=(c - gtyh) / D2, pobj=float(c @ xh))


def _net64(ws, bs, norm, u):
    z = (u.double() - norm[0].double()) / norm[1].double()
    z = torch.relu(z @ ws[0].T + bs[0])
    z = torch.relu(z @ ws[1].T + bs[1])
    return z @ ws[2].T + bs[2]


def exact(case, seed):
    if case["kind"] == "lp":
        if case["precision"] == "mixed":
            # how far its single-precision iterates are from these is the rounding of their storage, carried
            # through the line search: another order of one sum draws it anew (the spmv cases hold the products)
            return None
        e = _lp_exact(case, seed)
        return dict(x=e["x"], y=e["y"], lam=e["lam"], trials=None, accepted=None, restarts=None, omega=None, pobj=e["pobj"])
    if case["kind"] == "batch":
        es = [_lp_exact(dict(c, trials=case["trials"]), seed * 997 + i) for i, c in enumerate(_members(case))]
        return dict(x=torch.cat([e["x"] for e in es]), y=torch.cat([e["y"] for e in es]), lam=torch.cat([e["lam"] for e in es]),
                    accepted=None, restarts=None)
    if case["kind"] == "spmv":
        d = _lp_data(case, seed)
        t = torch.float64 if case["precision"] == "fp64" else torch.float32
        g = _gen(seed, 1)
        x = torch.randn(d["n"], generator=g, device="cuda", dtype=t).cpu().numpy().astype(np.float64)
        y = torch.randn(d["m"], generator=g, device="cuda", dtype=t).cpu().numpy().astype(np.float64)
        return dict(gx=np.bincount(d["row"], weights=d["val"] * x[d["col"]], minlength=d["m"]),
                    gty=np.bincount(d["col"], weights=d["val"] * y[d["row"]], minlength=d["n"]))
    if case["kind"] == "project":
        v, f = (torch.as_tensor(a, device="cuda") for a in _vectors(case, seed))
        return _cone_projection(case["cone"], v, f).cpu().numpy()
    ws, bs, norm, u, t = _net_data(case, seed)
    ps = [p.double() for pair in zip(ws, bs) for p in pair]
    if case["kind"] == "predict":
        return _net64(ps[0::2], ps[1::2], norm, u) * norm[3].double() + norm[2].double()
    ms, vs, losses = [torch.zeros_like(p) for p in ps], [torch.zeros_like(p) for p in ps], []
    for step, at in enumerate(range(0, len(u), case["batch"]), 1):
        ps = [p.detach().requires_grad_() for p in ps]
        want = (t[at:at + case["batch"]].double() - norm[2].double()) / norm[3].double()
        loss = (_net64(ps[0::2], ps[1::2], norm, u[at:at + case["batch"]]) - want).square().mean()
        losses.append(float(loss))
        with torch.no_grad():
            grads = torch.autograd.grad(loss, ps)
            ms = [0.9 * q + 0.1 * g for q, g in zip(ms, grads)]
            vs = [0.999 * q + 0.001 * g * g for q, g in zip(vs, grads)]
            ps = [p - 1e-3 * (q / (1 - 0.9 ** step)) / ((r / (1 - 0.999 ** step)).sqrt() + 1e-8) for p, q, r in zip(ps, ms, vs)]
    return dict(losses=np.array(losses), params=torch.cat([p.detach().reshape(-1) for p in ps]))

"""The work this library is used for, as cases that can be timed.

Each case is one call of a public entry point (paper_1502_07770_amd.binding) with the
inputs, weights and, where a program would keep them, the plans and the solver it holds.
``listed()`` names twelve of them, ``draw()`` gives others of the same ranges, and
``exact()`` solves a case again in 64 bits with plain torch: the message passing on sorted
breakpoint arrays, all chains (or trees) of a batch side by side.
"""
import math

import numpy as np
import torch

from paper_1502_07770_amd import binding

DEV = "cuda" if torch.cuda.is_available() else "cpu"


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # A handful of short signals in double precision, the smallest call: its time is latency.
        dict(name="prox_64x256_f64", kind="prox", dim=1, rows=64, cols=256, dtype="f64", edge_w=False, w=0.5),
        # Every row and every column of one large image in one launch, the plan tuned once per shape: the
        # library's headline, one step of any splitting method over the image.
        dict(name="prox_rows_cols_4096_f32", kind="both", rows=4096, cols=4096, dtype="f32", w=0.1),
        # A differentiable TV layer over a large batch of signals with learned edge weights: forward and backward.
        dict(name="grad_rows_65536x1024_f32", kind="grad", dim=1, rows=65536, cols=1024, dtype="f32"),
        # The same layer along the other axis of an odd-sized image.
        dict(name="grad_cols_3001x1111_f32", kind="grad", dim=0, rows=3001, cols=1111, dtype="f32"),
        # Weighted data terms and asymmetric edge weights on the rows of a large image.
        dict(name="dp_rows_4096_f32", kind="dp", dim=1, rows=4096, cols=4096, dtype="f32", w=0.1),
        # Impulse noise: TV-l1 on a large batch of signals.
        dict(name="l1_rows_65536x1024_f32", kind="l1", dim=1, rows=65536, cols=1024, dtype="f32", w=0.55, c=1.0),
        # Denoising an ordinary image to a fixed iteration count.
        dict(name="tv2d_512_f32", kind="tv2d", rows=512, cols=512, dtype="f32", lam=0.1, iters=200, tol=0.0, tuned=False),
        # The same in double precision on a small odd-sized image.
        dict(name="tv2d_203x317_f64", kind="tv2d", rows=203, cols=317, dtype="f64", lam=0.1, iters=40, tol=0.0, tuned=False),
        # A large image to a duality gap, with a solver that is kept and tuned once.
        dict(name="tv2d_4096_f32_gap", kind="tv2d", rows=4096, cols=4096, dtype="f32", lam=0.1, iters=500, tol=1e-5, tuned=True),
        # A set of images of different sizes and weights, each to its own duality gap.
        dict(name="tv2d_batch_24_f32", kind="batch", images=24, side_lo=64, side_hi=1024, dtype="f32", tol=1e-4),
        # Trees with quadratic and absolute data terms.
        dict(name="tree_16384x256_f32", kind="tree", trees=16384, nodes=256, dtype="f32"),
        # Stereo-like rows: sampled matching costs with a truncated pairwise term.
        dict(name="nc_rows_375x450x32_f32", kind="nc", rows=375, cols=450, levels=32, dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi, most):
    """Two log-uniform sides whose product is at most `most`."""
    while True:
        r, c = _log_int(rng, lo, hi), _log_int(rng, lo, hi)
        if r * c <= most:
            return r, c


def draw(rng):
    kind = rng.choice(["prox", "prox", "both", "grad", "grad", "dp", "l1", "tv2d", "tv2d", "batch", "tree", "nc"])
    dtype = rng.choice(["f32", "f32", "f32", "f64"])
    if kind == "prox":
        r, c = _sides(rng, 32, 65536, 1 << 24)
        return dict(kind=kind, dim=rng.choice([0, 1]), rows=r, cols=c, dtype=dtype, edge_w=rng.random() < 0.5,
                    w=round(rng.uniform(0.05, 0.6), 4))
    if kind == "both":
        r, c = _sides(rng, 64, 6000, 1 << 24)
        return dict(kind=kind, rows=r, cols=c, dtype=dtype, w=round(rng.uniform(0.05, 0.3), 4))
    if kind == "grad":
        r, c = _sides(rng, 64, 30000, 1 << 24)
        return dict(kind=kind, dim=rng.choice([0, 1]), rows=r, cols=c, dtype=dtype)
    if kind == "dp":
        r, c = _sides(rng, 64, 8192, 1 << 23)
        return dict(kind=kind, dim=rng.choice([0, 1]), rows=r, cols=c, dtype=dtype, w=round(rng.uniform(0.05, 0.3), 4))
    if kind == "l1":
        r, c = _sides(rng, 64, 16384, 1 << 22)
        return dict(kind=kind, dim=rng.choice([0, 1]), rows=r, cols=c, dtype=dtype, w=round(rng.uniform(0.3, 0.8), 4),
                    c=round(rng.uniform(0.5, 1.5), 4))
    if kind == "tv2d":
        r, c = _sides(rng, 64, 2048, 1 << 21)
        tol = rng.choice([0.0, 1e-4, 1e-5])
        return dict(kind=kind, rows=r, cols=c, dtype=dtype, lam=round(rng.uniform(0.03, 0.25), 4),
                    iters=rng.randint(20, 60) if tol == 0.0 else 500, tol=tol, tuned=rng.random() < 0.3)
    if kind == "batch":
        lo = rng.randint(48, 128)
        return dict(kind=kind, images=rng.randint(3, 24), side_lo=lo, side_hi=lo + rng.randint(100, 700), dtype=dtype,
                    tol=rng.choice([1e-4, 1e-5]))
    if kind == "tree":
        return dict(kind=kind, trees=_log_int(rng, 64, 16384), nodes=rng.randint(40, 256), dtype=dtype)
    return dict(kind="nc", rows=_log_int(rng, 40, 375), cols=_log_int(rng, 60, 450), levels=rng.randint(12, 40), dtype=dtype)


def _dt(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


# ---------------------------------------------------------------------------
# Inputs, made on the device from the seed
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _signals(C, n, g, sigma=0.1):
    """Piecewise-constant chains: a new level with probability 1/20 per node, levels U[0, 1], plus N(0, sigma^2)."""
    run = (torch.rand(C, n, generator=g, device=DEV) < 0.05).to(torch.int32).cumsum(1)
    lev = torch.rand(C, n + 1, generator=g, device=DEV)
    y = lev.gather(1, run.long())
    if sigma > 0:
        y = y + sigma * torch.randn(C, n, generator=g, device=DEV)
    return y


def _image(H, W, g, sigma=0.1):
    """30 rectangles and disks of intensity U[0, 1] over zero, plus N(0, sigma^2)."""
    p = torch.rand(30, 6, generator=g, device=DEV).tolist()
    img = torch.zeros(H, W, device=DEV)
    rr = torch.arange(H, device=DEV, dtype=torch.float32)[:, None]
    cc = torch.arange(W, device=DEV, dtype=torch.float32)[None, :]
    m = min(H, W)
    for kind, inten, cy, cx, a, b in p:
        cy, cx = cy * H, cx * W
        if kind < 0.5:
            h, w = H / 20 + a * (H / 3 - H / 20), W / 20 + b * (W / 3 - W / 20)
            r0, r1 = max(int(cy - h / 2), 0), min(int(cy + h / 2) + 1, H)
            c0, c1 = max(int(cx - w / 2), 0), min(int(cx + w / 2) + 1, W)
            img[r0:r1, c0:c1] = inten
        else:
            rad = m / 40 + a * (m / 6 - m / 40)
            img.masked_fill_((rr - cy) ** 2 + (cc - cx) ** 2 <= rad * rad, inten)
    return img + sigma * torch.randn(H, W, generator=g, device=DEV)


def _weights(shape, g, lo=0.1, hi=1.0):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device=DEV)


def _forest(T, n, g):
    """T post-order trees of n nodes: a node adopts 0 to 3 of the most recent pending subtrees, the last one all.
    Returns the parents within each tree, (T, n), -1 at the roots."""
    u = torch.rand(n, T, generator=g, device=DEV)
    want = (u > 0.4).long() + (u > 0.7).long() + (u > 0.9).long()
    parent = torch.full((n, T), -1, dtype=torch.int64, device=DEV)
    stack = torch.zeros(n + 1, T, dtype=torch.int64, device=DEV)
    sp = torch.zeros(T, dtype=torch.int64, device=DEV)
    for j in range(n - 1):
        k = torch.minimum(want[j], sp)
        for r in range(3):
            on = k > r
            top = stack.gather(0, (sp - 1).clamp(min=0)[None])[0]
            old = parent.gather(0, top[None])[0]
            parent.scatter_(0, top[None], torch.where(on, j, old)[None])
            sp = sp - on.long()
        stack.scatter_(0, sp[None], torch.full((1, T), j, dtype=torch.int64, device=DEV))
        sp = sp + 1
    parent[:n - 1] = torch.where(parent[:n - 1] < 0, n - 1, parent[:n - 1])
    return parent.t().contiguous()


def _l1_data(case, g):
    """Chains along `dim` of clean piecewise-constant signals with a quarter of the samples set to 0 or 1."""
    C, n = (case["rows"], case["cols"]) if case["dim"] == 1 else (case["cols"], case["rows"])
    y = _signals(C, n, g, sigma=0.0)
    hit = torch.rand(C, n, generator=g, device=DEV) < 0.25
    y = torch.where(hit, (torch.rand(C, n, generator=g, device=DEV) < 0.5).float(), y)
    return (y if case["dim"] == 1 else y.t().contiguous())


def _along(case, g):
    """Piecewise-constant noisy signals along `dim` of a rows x cols tensor."""
    if case["dim"] == 1:
        return _signals(case["rows"], case["cols"], g)
    return _signals(case["cols"], case["rows"], g).t().contiguous()


def _inputs(case, seed):
    """The case's inputs in the precision it runs in."""
    g, dt, kind = _gen(seed), _dt(case), case["kind"]
    d = {}
    if kind == "prox":
        d["y"] = _along(case, g).to(dt)
        if case["edge_w"]:
            d["w"] = (case["w"] * _weights(d["y"].shape, g, 0.2, 1.8)).to(dt)
    elif kind == "both":
        d["y"] = _image(case["rows"], case["cols"], g).to(dt)
    elif kind == "grad":
        d["y"] = _along(case, g).to(dt)
        d["w"] = _weights(d["y"].shape, g).to(dt)
        d["g"] = torch.randn(d["y"].shape, generator=g, device=DEV).to(dt)
    elif kind == "dp":
        f = _image(case["rows"], case["cols"], g)
        a = _weights(f.shape, g, 0.5, 2.0)
        d["a"], d["b"] = a.to(dt), (a * f).to(dt)
        d["wm"] = (-case["w"] * _weights(f.shape, g, 0.5, 1.5)).to(dt)
        d["wp"] = (case["w"] * _weights(f.shape, g, 0.5, 1.5)).to(dt)
    elif kind == "l1":
        d["y"] = _l1_data(case, g).to(dt)
        d["d"] = d["y"].clone()
    elif kind == "tv2d":
        d["f"] = _image(case["rows"], case["cols"], g).to(dt)
    elif kind == "batch":
        n = case["images"]
        span = case["side_hi"] - case["side_lo"] + 1
        u = np.random.RandomState(n * 1009 + case["side_lo"] * 31 + case["side_hi"]).rand(n, 4)  # sizes do not follow the seed
        d["shapes"] = [(case["side_lo"] + int(v[0] * span), case["side_lo"] + int(v[1] * span)) for v in u]
        d["lams"] = [0.02 + 0.28 * float(v[2]) for v in u]
        d["images"] = [_image(h, w, g, 0.05 + 0.15 * float(v[3])).to(dt) for (h, w), v in zip(d["shapes"], u)]
    elif kind == "tree":
        T, n = case["trees"], case["nodes"]
        d["parent"] = _forest(T, n, g)
        a = _weights((T, n), g, 0.3, 2.0)
        d["a"], d["b"] = a.to(dt), (a * torch.randn(T, n, generator=g, device=DEV)).to(dt)
        on = torch.rand(T, n, generator=g, device=DEV) < 0.7
        d["c"] = (on * torch.rand(T, n, generator=g, device=DEV)).to(dt)
        d["d"] = torch.randn(T, n, generator=g, device=DEV).to(dt)
        d["wm"] = (-0.8 * torch.rand(T, n, generator=g, device=DEV)).to(dt)
        d["wp"] = (0.8 * torch.rand(T, n, generator=g, device=DEV)).to(dt)
    else:
        H, W, D = case["rows"], case["cols"], case["levels"]
        disp = _image(H, W, g, 0.0) * (D - 1)
        lev = torch.arange(D, device=DEV, dtype=torch.float32)
        cost = (lev - disp[:, :, None]).abs().clamp(max=4.0) + 0.1 * torch.randn(H, W, D, generator=g, device=DEV)
        bad = torch.rand(H, W, 1, generator=g, device=DEV) < 0.1
        cost = torch.where(bad, 4.0 * torch.rand(H, W, D, generator=g, device=DEV), cost).double()
        steep = torch.full((H, W, 1), 10.0, device=DEV, dtype=torch.float64)
        d["uslope"] = torch.cat([-steep, cost[:, :, 1:] - cost[:, :, :-1], steep], 2).reshape(-1).to(dt)
        d["ulam"] = lev.repeat(H * W).to(dt)
        d["coff"] = torch.arange(H + 1, device=DEV, dtype=torch.int64) * W
        d["uoff"] = torch.arange(H * W + 1, device=DEV, dtype=torch.int64) * D
        d["w"] = torch.full((H * W,), 0.6, device=DEV, dtype=dt)
        d["C"] = torch.full((H * W,), 2.0, device=DEV, dtype=dt)
    return d


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind == "both":
        binding.autotune_chain_prox([(s["y"], 1), (s["y"], 0)], case["w"])
    elif kind == "grad":
        s["y"].requires_grad_(True)
        s["w"].requires_grad_(True)
    elif kind == "tv2d":
        s["solver"] = binding.Tv2dSolver(case["rows"], case["cols"], _dt(case), s["f"].device)
        if case["tuned"]:
            s["solver"].autotune(s["f"], case["lam"])
    elif kind == "tree":
        T, n = case["trees"], case["nodes"]
        base = torch.arange(T, device=DEV, dtype=torch.int64)[:, None] * n
        s["gparent"] = torch.where(s["parent"] >= 0, s["parent"] + base, -1).reshape(-1)
        s["offsets"] = torch.arange(T + 1, device=DEV, dtype=torch.int64) * n
        for k in ("a", "b", "c", "d", "wm", "wp"):
            s[k] = s[k].reshape(-1)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "prox":
        return binding.chain_prox(s["y"], s["w"] if case["edge_w"] else case["w"], dim=case["dim"])
    if kind == "both":
        return binding.chain_prox_multi([(s["y"], 1), (s["y"], 0)], case["w"])
    if kind == "grad":
        x = binding.prox(s["y"], s["w"], dim=case["dim"])
        gy, gw = torch.autograd.grad(x, (s["y"], s["w"]), s["g"])
        return x.detach(), gy, gw
    if kind == "dp":
        return binding.chain_dp(s["b"], s["wm"], s["wp"], a=s["a"], dim=case["dim"])
    if kind == "l1":
        return binding.chain_prox_l1(s["y"], s["d"], case["w"], case["c"], dim=case["dim"])
    if kind == "tv2d":
        x, info = s["solver"].solve(s["f"], case["lam"], max_iter=case["iters"], gap_every=4 if case["tol"] > 0 else 10,
                                    gap_tol=case["tol"])
        return x, info["iters"]
    if kind == "batch":
        xs, infos = binding.tv2d_batched(s["images"], s["lams"], max_iter=300, gap_every=2, gap_tol=case["tol"])
        return xs, [i["iters"] for i in infos]
    if kind == "tree":
        return binding.tree_dp(s["gparent"], s["offsets"], s["b"], s["wm"], s["wp"], a=s["a"], c=s["c"], d=s["d"])
    return binding.chain_nc(s["coff"], s["uoff"], s["ulam"], s["uslope"], s["w"], s["C"])


def work(case):
    """Bytes of the inputs and outputs once; about 15 operations per node and message update.  A 2D iteration reads
    and writes the state once (32 bytes per pixel in FP32); solves to a gap of 1e-4 (1e-5) take about 6 (12)."""
    kind, e = case["kind"], 8 if case["dtype"] == "f64" else 4
    if kind == "batch":
        side = 0.5 * (case["side_lo"] + case["side_hi"])
        px, it = case["images"] * side * side, 6 if case["tol"] >= 1e-4 else 12
        return dict(bytes=8 * e * it * px, flops=40.0 * it * px)
    if kind == "tree":
        n = case["trees"] * case["nodes"]
        return dict(bytes=n * (7 * e + 8), flops=60.0 * n)
    n = case["rows"] * case["cols"]
    if kind == "prox":
        return dict(bytes=n * e * (3 if case["edge_w"] else 2), flops=15.0 * n)
    if kind == "both":
        return dict(bytes=4.0 * n * e, flops=30.0 * n)
    if kind == "grad":
        return dict(bytes=7.0 * n * e, flops=20.0 * n)
    if kind == "dp":
        return dict(bytes=5.0 * n * e, flops=20.0 * n)
    if kind == "l1":
        return dict(bytes=3.0 * n * e, flops=25.0 * n)
    if kind == "tv2d":
        it = case["iters"] if case["tol"] == 0.0 else 6 if case["tol"] >= 1e-4 else 12
        return dict(bytes=8.0 * n * e * it, flops=40.0 * n * it)
    return dict(bytes=n * e * (2 * case["levels"] + 4), flops=20.0 * n * case["levels"])


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch.
#
# The derivative of a message is a non-decreasing function with sorted breakpoints
# (position l, change a of the slope, change b of the intercept), rows of (M, C) arrays for
# C problems side by side; unused rows hold l = +inf.  It is `lo` left of its breakpoints
# and `hi` right of them.
# ---------------------------------------------------------------------------

def _rows(M, like):
    return torch.arange(M, device=like.device)[:, None]


def _shift(E, idx, keep):
    """E[idx] along the rows where keep, empty elsewhere."""
    out = []
    for k, t in enumerate(E):
        v = t.gather(0, idx.clamp(0, t.shape[0] - 1))
        out.append(torch.where(keep, v, math.inf if k == 0 else 0.0))
    return out


def _grow(E, extra):
    return [torch.cat([t, torch.full((extra,) + t.shape[1:], math.inf if k == 0 else 0.0, dtype=t.dtype, device=t.device)])
            for k, t in enumerate(E)]


def _put(E, row, vals, on=None):
    for t, v in zip(E, vals):
        v = v if on is None else torch.where(on, v, t.gather(0, row[None])[0])
        t.scatter_(0, row[None], v[None])


def _insert(E, n, l, b, on):
    """Adds the breakpoint (l, 0, b) where `on`."""
    M = E[0].shape[0]
    q = (E[0] <= l).sum(0)
    r = _rows(M, l)
    idx = torch.where((r > q) & on, r - 1, r)
    E = _shift(E, idx, r < n + on.long())
    _put(E, q.clamp(max=M - 1), (l, torch.zeros_like(l), b), on)
    return E, n + on.long()


def _scan(E, n, A0, B0):
    A, B = A0 + E[1].cumsum(0), B0 + E[2].cumsum(0)
    l = torch.where(torch.isinf(E[0]), 0.0, E[0])
    Ap, Bp = torch.cat([A0[None], A]), torch.cat([B0[None], B])  # the piece left of row j
    valid = _rows(E[0].shape[0], l) < n
    return Ap, Bp, l, torch.where(valid, A * l + B, math.inf), valid


def _root_of(E, Ap, Bp, p, n, v):
    """Where the function crosses v on the piece left of breakpoint p, kept between its neighbours."""
    M = E[0].shape[0]
    a, b = Ap.gather(0, p[None])[0], Bp.gather(0, p[None])[0]
    z = (v - b) / a
    right = torch.where(p < n, E[0].gather(0, p.clamp(max=M - 1)[None])[0], math.inf)
    left = torch.where(p > 0, E[0].gather(0, (p - 1).clamp(min=0)[None])[0], -math.inf)
    return torch.maximum(torch.minimum(z, right), left), a, b, right


def _step(E, n, a, b, c, d, lo0, hi0, lo, hi, l1):
    """Adds the unary a z - b + c sign(z - d) to the message with ends lo0, hi0 and clips it to [lo, hi].
    Returns the message, its size and the two crossings."""
    if int(n.max()) + 3 > E[0].shape[0]:
        E = _grow(E, 8)
    M = E[0].shape[0]
    r = _rows(M, lo)
    if l1:
        E, n = _insert(E, n, d, 2 * c, c > 0)
    A0, B0 = a, lo0 - b - c
    Ap, Bp, l, hr, valid = _scan(E, n, A0, B0)
    p = ((hr < lo) & valid).sum(0)
    zl, pa, pb, right = _root_of(E, Ap, Bp, p, n, lo)
    pj = p.clamp(max=M - 1)
    jump = (p < n) & (zl >= right)
    drop = p + jump.long()
    pa = torch.where(jump, Ap.gather(0, (pj + 1)[None])[0], pa)
    pb = torch.where(jump, Bp.gather(0, (pj + 1)[None])[0], pb)
    n = n - drop + 1
    E = _shift(E, r + drop - 1, r < n)
    E[0][0], E[1][0], E[2][0] = zl, pa, pb - lo
    Ap, Bp, l, hr, valid = _scan(E, n, torch.zeros_like(a), lo)
    keep = ((hr <= hi) & valid).sum(0).clamp(min=1)
    # lo = hi, or a first breakpoint whose jump passes hi: everything is cut at zl
    cut = hr[0] > hi
    z, pa, pb, _ = _root_of(E, Ap, Bp, torch.where(cut, 1, keep), n, hi)
    flat = cut | (pa <= 0)
    zr = torch.where(flat, zl, torch.maximum(z, zl))
    E = _shift(E, r.expand(M, a.shape[0]), r < keep)
    e1, e2 = -pa, hi - pb
    E[1][0], E[2][0] = torch.where(flat, 0.0, E[1][0]), torch.where(flat, hi - lo, E[2][0])
    n = torch.where(flat, 1, keep + 1)
    E = _shift(E, r.expand(M, a.shape[0]), r < n)
    _put(E, torch.where(flat, 0, keep), (torch.where(flat, zl, zr), torch.where(flat, E[1][0], e1), torch.where(flat, E[2][0], e2)))
    return E, n, zl, zr


def _empty(C, like):
    return [torch.full((8, C), math.inf if k == 0 else 0.0, dtype=torch.float64, device=like.device) for k in range(3)]


def _trim(E, n):
    m = int(n.max()) + 3
    return [t[:m].clone() for t in E] if m + 8 < E[0].shape[0] else E


def _zero(E, n, a, b, c, d, lo0, l1):
    """The zero of the message plus its unary (at a root)."""
    if l1:
        if int(n.max()) + 1 > E[0].shape[0]:
            E = _grow(E, 2)
        E, n = _insert(E, n, d, 2 * c, c > 0)
    Ap, Bp, l, hr, valid = _scan(E, n, a, lo0 - b - c)
    p = ((hr < 0) & valid).sum(0)
    return _root_of(E, Ap, Bp, p, n, torch.zeros_like(a))[0]


def _chains(b, wm, wp, a=None, c=None, d=None):
    """Exact chains in 64 bits; every argument (n, C), edge i joins nodes i and i + 1."""
    n, C = b.shape
    one, zero = torch.ones_like(b[0]), torch.zeros_like(b[0])
    L, U = torch.empty_like(b), torch.empty_like(b)
    E, m, lo0, hi0 = _empty(C, b), torch.zeros(C, dtype=torch.int64, device=b.device), zero, zero
    l1 = c is not None
    for i in range(n - 1):
        ai = one if a is None else a[i]
        ci, di = (c[i], d[i]) if l1 else (zero, zero)
        E, m, L[i], U[i] = _step(E, m, ai, b[i], ci, di, lo0, hi0, wm[i], wp[i], l1)
        lo0, hi0 = wm[i], wp[i]
        if i % 32 == 31:
            E = _trim(E, m)
    i = n - 1
    x = torch.empty_like(b)
    x[i] = _zero(E, m, one if a is None else a[i], b[i], c[i] if l1 else zero, d[i] if l1 else zero, lo0, l1)
    for i in range(n - 2, -1, -1):
        x[i] = torch.maximum(torch.minimum(x[i + 1], U[i]), L[i])
    return x


def _prox(y, w):
    """TV prox of every column of y; w (n, C) or a number."""
    w = w if isinstance(w, torch.Tensor) else torch.full_like(y, w)
    return _chains(y, -w, w)


def _adjoint(x, g):
    """Gradients by the runs of equal values of every column."""
    n, C = x.shape
    first = torch.ones(n, C, dtype=torch.bool, device=x.device)
    first[1:] = x[1:] != x[:-1]
    rid = first.long().cumsum(0) - 1
    tot = torch.zeros_like(x).scatter_add_(0, rid, g)
    cnt = torch.zeros_like(x).scatter_add_(0, rid, torch.ones_like(g))
    gy = (tot / cnt.clamp(min=1)).gather(0, rid)
    gw = torch.zeros_like(x)
    gw[:-1] = torch.sign(x[1:] - x[:-1]) * (gy[:-1] - gy[1:])
    return gy, gw


def _rof(f, lam, iters):
    """The accelerated primal-dual iterate of the row and column splitting after `iters` steps."""
    x, y, xb, tau = f.clone(), torch.zeros_like(f), f.clone(), 1.0
    for _ in range(iters):
        eta = y + xb / tau
        y = eta - _prox(eta, lam)
        b = (tau * f + x - tau * y) / (1 + tau)
        xn = _prox(b.t().contiguous(), lam * tau / (1 + tau)).t()
        th = 1 / math.sqrt(1 + 2 * tau)
        x, xb, tau = xn, xn + th * (xn - x), th * tau
    return x


def _trees(parent, a, b, c, d, wm, wp):
    """Exact trees in 64 bits; every argument (n, T), parents within the tree, post-order."""
    n, T = b.shape
    dev = b.device
    L, U, X = torch.empty_like(b), torch.empty_like(b), torch.empty_like(b)
    S, M = 8, 8
    st = [torch.full((S, M, T), math.inf if k == 0 else 0.0, dtype=torch.float64, device=dev) for k in range(3)]
    scnt, sfor, slo, shi = (torch.zeros(S, T, dtype=t, device=dev) for t in (torch.int64, torch.int64, torch.float64, torch.float64))
    sp = torch.zeros(T, dtype=torch.int64, device=dev)
    ar = torch.arange(T, device=dev)
    for j in range(n):
        E, m = _empty(T, b), torch.zeros(T, dtype=torch.int64, device=dev)
        lo0, hi0 = torch.zeros(T, dtype=torch.float64, device=dev), torch.zeros(T, dtype=torch.float64, device=dev)
        while True:
            top = (sp - 1).clamp(min=0)
            on = (sp > 0) & (sfor[top, ar] == j)
            if not bool(on.any()):
                break
            child = [torch.where(on, t[top, :, ar].t(), math.inf if k == 0 else 0.0) for k, t in enumerate(st)]
            both = [torch.cat([u, v]) for u, v in zip(E, child)]
            l, order = both[0].sort(dim=0, stable=True)
            E = [l, both[1].gather(0, order), both[2].gather(0, order)]
            m = m + torch.where(on, scnt[top, ar], 0)
            E = [t[:max(8, int(m.max()) + 3)].clone() for t in E]
            lo0, hi0 = lo0 + torch.where(on, slo[top, ar], 0.0), hi0 + torch.where(on, shi[top, ar], 0.0)
            sp = sp - on.long()
        if j == n - 1:
            X[j] = _zero(E, m, a[j], b[j], c[j], d[j], lo0, True)
            break
        E, m, L[j], U[j] = _step(E, m, a[j], b[j], c[j], d[j], lo0, hi0, wm[j], wp[j], True)
        k = int(m.max())
        if k > M:
            st = [torch.cat([t, torch.full((S, k + 8 - M, T), math.inf if q == 0 else 0.0, dtype=torch.float64, device=dev)], 1)
                  for q, t in enumerate(st)]
            M = k + 8
        if int(sp.max()) + 1 > S:
            st = [torch.cat([t, torch.zeros(8, M, T, dtype=torch.float64, device=dev)]) for t in st]
            scnt, sfor, slo, shi = (torch.cat([t, torch.zeros(8, T, dtype=t.dtype, device=dev)]) for t in (scnt, sfor, slo, shi))
            S += 8
        E = _grow(E, max(0, M - E[0].shape[0]))
        for q in range(3):
            st[q][sp, :, ar] = E[q][:M].t()
        scnt[sp, ar], sfor[sp, ar], slo[sp, ar], shi[sp, ar] = m, parent[j], wm[j], wp[j]
        sp = sp + 1
    for j in range(n - 2, -1, -1):
        X[j] = torch.maximum(torch.minimum(X.gather(0, parent[j][None])[0], U[j]), L[j])
    return X


def exact(case, seed):
    """What run() returns, in 64 bits; None where that takes too long or (argmins of non-convex energies) has no
    plain form."""
    kind = case["kind"]
    if kind in ("nc", "batch"):
        return None
    if kind == "tv2d" and (case["tol"] > 0 or case["iters"] * (case["rows"] + case["cols"]) > 21000):
        return None
    if kind in ("prox", "grad") and (case["cols"] if case["dim"] == 1 else case["rows"]) > 20000:
        return None
    s = _inputs(case, seed)
    v = {k: t.double() for k, t in s.items() if torch.is_tensor(t) and t.is_floating_point()}
    if case.get("dim") == 1:
        v = {k: t.t().contiguous() for k, t in v.items()}
    back = (lambda t: t.t().contiguous()) if case.get("dim") == 1 else (lambda t: t)
    if kind == "prox":
        return back(_prox(v["y"], v["w"] if case["edge_w"] else case["w"]))
    if kind == "both":
        return [_prox(v["y"].t().contiguous(), case["w"]).t().contiguous(), _prox(v["y"], case["w"])]
    if kind == "grad":
        x = _prox(v["y"], v["w"])
        gy, gw = _adjoint(x, v["g"])
        return back(x), back(gy), back(gw)
    if kind == "dp":
        return back(_chains(v["b"], v["wm"], v["wp"], a=v["a"]))
    if kind == "l1":
        w = torch.full_like(v["y"], case["w"])
        return back(_chains(v["y"], -w, w, c=torch.full_like(w, case["c"]), d=v["d"]))
    if kind == "tv2d":
        return _rof(v["f"], case["lam"], case["iters"]), None
    p = s["parent"].t().contiguous()
    t = {k: v[k].t().contiguous() for k in ("a", "b", "c", "d", "wm", "wp")}
    return _trees(p, t["a"], t["b"], t["c"], t["d"], t["wm"], t["wp"]).t().reshape(-1)

"""The work that a user of this library has it do, as timed cases.

A case is one system (or a batch of systems) and one call or short chain of calls through the
public entry points of ``paper_2212_11675_amd``: the two products, the binary64 PC-LSQR solve,
the precision form (binary32 coefficients with binary64 residual correction), the variance
solve with constraint rows, the differentiable least-squares solve forward and backward, and
the batched multi-right-hand-side solves.  Sizes run from a system whose time is launches
(6e4 rows) to the widths of the largest benchmark workload (100,000 attitude knots per axis,
10,000 instrumental columns) at 1e8 rows, the most that leaves room for several systems at
once on one GPU.  Inputs are drawn on the GPU with the structure of the paper's Section 3 (the
distributions of ``synth``): rows sorted by star, N(0, 1) coefficients, attitude start uniform,
six distinct ascending instrumental columns, x_true ~ N(0, 1), noise N(0, 1e-3^2).
"""
from __future__ import annotations

import math

import torch

from paper_2212_11675_amd import autograd, gsr

NOISE = 1e-3     # standard deviation of the observation noise
CHUNK = 4 << 20  # rows handled at a time by the generator and by the plain torch reference


# ---- the cases --------------------------------------------------------------------------

def listed():
    return [
        # y = A x and x = A^T y on a small system (1,000 stars x 60 observations, the smallest
        # workload): what a caller pays per product when launches dominate
        dict(name="products_60k", kind="products", stars=1000, obs_lo=60, obs_hi=60, n_dfa=1000,
             n_instr=500, f32=False),
        # the same two products with the binary32 coefficient copy, uneven observation counts
        # and sizes off every power of two
        dict(name="products_f32_1m", kind="products", stars=31_337, obs_lo=10, obs_hi=60,
             n_dfa=3001, n_instr=1999, f32=True),
        # the products at the benchmark's 2e7-row size (a residual or a gradient step of a
        # caller's own iteration)
        dict(name="products_20m", kind="products", stars=1_000_000, obs_lo=20, obs_hi=20,
             n_dfa=30_000, n_instr=6000, f32=False),
        # one small solve at a fixed iteration count: the latency-bound end
        dict(name="solve_60k", kind="solve", stars=1000, obs_lo=60, obs_hi=60, n_dfa=1000,
             n_instr=500, iters=100),
        # the benchmark's 2e7-row system
        dict(name="solve_20m", kind="solve", stars=1_000_000, obs_lo=20, obs_hi=20, n_dfa=30_000,
             n_instr=6000, iters=20),
        # half of the largest benchmark system, at its full attitude and instrumental widths
        dict(name="solve_100m", kind="solve", stars=2_500_000, obs_lo=40, obs_hi=40,
             n_dfa=100_000, n_instr=10_000, iters=10),
        # more instrumental columns than one block keeps in LDS (the tests' 11,000)
        dict(name="solve_wide_4m", kind="solve", stars=115_001, obs_lo=10, obs_hi=60, n_dfa=11_500,
             n_instr=11_000, iters=20),
        # the precision form to a tolerance, as the benchmark sets it
        dict(name="refine_20m", kind="refine", stars=1_000_000, obs_lo=20, obs_hi=20,
             n_dfa=30_000, n_instr=6000),
        # constraint rows over a tenth of the stars, an odd mid-sized system solved to a
        # tolerance
        dict(name="con_3m", kind="con", stars=88_889, obs_lo=10, obs_hi=60, n_dfa=8887,
             n_instr=3001),
        # forward and backward through the differentiable least-squares solve (new coefficients
        # every step, as in a training loop)
        dict(name="grad_2m", kind="grad", stars=100_003, obs_lo=20, obs_hi=20, n_dfa=5003,
             n_instr=1500),
        # 16 systems of mixed size, eight right-hand sides each, fixed iterations
        dict(name="batch_k8_12m", kind="batch", n_sys=16, s_lo=1000, s_hi=100_000, n_instr=500,
             k=8, iters=20, tol=0.0),
        # many small systems with two right-hand sides each, every pair to its own tolerance
        dict(name="batch_k2_tol_2m", kind="batch", n_sys=64, s_lo=200, s_hi=2000, n_instr=100,
             k=2, iters=500, tol=1e-10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["products", "products", "solve", "solve", "solve", "refine", "con", "grad",
                       "batch", "batch"])
    if kind == "batch":
        s_lo = _log_int(rng, 200, 1000)
        c = dict(kind="batch", n_sys=rng.choice([3, 8, 16, 33, 64]), s_lo=s_lo,
                 s_hi=s_lo * rng.randint(2, 20), n_instr=_log_int(rng, 50, 500),
                 k=rng.choice([1, 2, 4, 8]), iters=rng.randint(10, 40), tol=0.0)
        if rng.random() < 0.4:
            c.update(iters=500, tol=1e-10)
        return c
    rows_lo, rows_hi = dict(products=(6e4, 2e7), solve=(6e4, 1e8), refine=(1e6, 2e7),
                            con=(1e5, 1e7), grad=(1e5, 2e6))[kind]
    lo, hi = rng.choice([(20, 20), (40, 40), (60, 60), (10, 60)])
    rows = math.exp(rng.uniform(math.log(rows_lo), math.log(rows_hi)))
    stars = max(1000, int(rows / (0.5 * (lo + hi))))
    rows = stars * 0.5 * (lo + hi)
    c = dict(kind=kind, stars=stars, obs_lo=lo, obs_hi=hi,
             n_dfa=_log_int(rng, 200, max(201, min(100_000, rows / 60))),
             n_instr=_log_int(rng, 100, max(101, min(10_000, rows / 100))))
    if kind == "products":
        c["f32"] = rng.random() < 0.4
    if kind == "solve":
        if rows > 2e6 and rng.random() < 0.2:
            c["n_instr"] = rng.randint(10_241, 20_000)
        c["iters"] = int(min(40, max(10, 4e8 / rows)))
        if rows < 1e7 and rng.random() < 0.3:  # with the variance estimate
            c.update(var=True, iters=rng.randint(10, 20))
    return c


# ---- inputs -----------------------------------------------------------------------------

def _gen(seed, stream=0):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + int(stream))


def _system(stars, lo, hi, n_dfa, n_instr, gen):
    """One system's arrays in the library's row layout (CUDA tensors)."""
    # every count of lo..hi equally often (the row count is the case's, not the seed's), stars
    # in random order
    counts = lo + torch.randperm(stars, device="cuda", generator=gen) % (hi - lo + 1)
    m = int(counts.sum())
    star = torch.repeat_interleave(torch.arange(stars, dtype=torch.int32, device="cuda"), counts)
    vals = torch.empty(24 * m, dtype=torch.float64, device="cuda")
    att = torch.empty(m, dtype=torch.int32, device="cuda")
    instr = torch.empty(6 * m, dtype=torch.int32, device="cuda")
    six = torch.arange(6, device="cuda", dtype=torch.int32)
    for r0 in range(0, m, CHUNK):
        r1 = min(m, r0 + CHUNK)
        vals[24 * r0:24 * r1].normal_(generator=gen)
        att[r0:r1].random_(0, n_dfa - 3, generator=gen)
        # six ascending order statistics of n_instr - 5 places, spread to distinct columns
        e = torch.empty(r1 - r0, 7, dtype=torch.float64, device="cuda").exponential_(generator=gen)
        u = torch.cumsum(e, 1)
        place = (u[:, :6] / u[:, 6:] * (n_instr - 5)).to(torch.int32).clamp_(max=n_instr - 6)
        instr[6 * r0:6 * r1] = (place + six).reshape(-1)
    return dict(m=m, stars=stars, n_dfa=n_dfa, n_instr=n_instr,
                n=5 * stars + 3 * n_dfa + n_instr + 1, vals=vals, star=star, att=att, instr=instr)


def _normal(count, gen, scale=1.0):
    return torch.empty(count, dtype=torch.float64, device="cuda").normal_(0.0, scale,
                                                                          generator=gen)


def _one_system(case, seed):
    gen = _gen(seed)
    s = _system(case["stars"], case["obs_lo"], case["obs_hi"], case["n_dfa"], case["n_instr"], gen)
    return s, gen


def _rhs(s, gen):
    x_true = _normal(s["n"], gen)
    return _times(s, x_true) + _normal(s["m"], gen, NOISE)


def _constraints(case, s, gen):
    """Six reference-frame-like rows, two astrometric unknowns of every selected star each, and
    their right-hand side."""
    prim = torch.nonzero(torch.rand(case["stars"], device="cuda", generator=gen) < 0.1).reshape(-1)
    per = 2 * prim.numel()
    ptr = torch.arange(7, device="cuda", dtype=torch.int64) * per
    col = torch.cat([torch.stack([5 * prim + a, 5 * prim + a + 1], 1).reshape(-1)
                     for a in (1, 1, 1, 3, 3, 3)]).to(torch.int64)
    return (ptr, col, _normal(6 * per, gen)), _normal(6, gen)


def _batch_stars(case):
    n = case["n_sys"]
    lo, hi = math.log(case["s_lo"]), math.log(case["s_hi"])
    # log-spaced sizes in a scattered order
    return [int(round(math.exp(lo + (hi - lo) * ((i * 7919) % n) / max(1, n - 1))))
            for i in range(n)]


def _batch_systems(case, seed):
    gen = _gen(seed)
    out = []
    for stars in _batch_stars(case):
        s = _system(stars, 10, 60, max(4, stars // 10), case["n_instr"], gen)
        out.append((s, torch.stack([_rhs(s, gen) for _ in range(case["k"])], 1)))
    return out


def _dims(s):
    return gsr.make_dims(s["m"], s["stars"], s["n_dfa"], s["n_instr"])


def _open(s, **kw):
    return gsr.gsr_lsqr_setup(_dims(s), s["vals"], s["star"], s["att"], s["instr"],
                              allow_empty_cols=True, **kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        systems = _batch_systems(case, seed)
        ro = [0]
        for s, _ in systems:
            ro.append(ro[-1] + s["m"])
        cat = {k: torch.cat([s[k] for s, _ in systems]) for k in ("vals", "star", "att", "instr")}
        b = gsr.gsr_batch_setup([_dims(s) for s, _ in systems], ro, cat["vals"], cat["star"],
                                cat["att"], cat["instr"], case["k"], allow_empty_cols=True)
        rhs = torch.cat([r.reshape(-1) for _, r in systems])
        opts = gsr.solve_opts(itnlim=case["iters"], fixed_iters=case["tol"] == 0.0,
                              atol=case["tol"], btol=case["tol"])
        return dict(case=case, b=b, rhs=rhs, opts=opts,
                    x=torch.empty(b.n * b.k, dtype=torch.float64, device="cuda"))
    s, gen = _one_system(case, seed)
    if kind == "products":
        return dict(case=case, h=_open(s, build_f32=case["f32"]), x=_normal(s["n"], gen),
                    y=_normal(s["m"], gen), ax=torch.empty(s["m"], dtype=torch.float64, device="cuda"),
                    aty=torch.empty(s["n"], dtype=torch.float64, device="cuda"))
    b = _rhs(s, gen)
    if kind == "grad":
        st = autograd.Structure(s["star"], s["att"], s["instr"], s["stars"], s["n_dfa"],
                                s["n_instr"])
        return dict(case=case, structure=st, vals=s["vals"].requires_grad_(True),
                    b=b.requires_grad_(True), x_ref=_normal(s["n"], gen))
    x = torch.empty(s["n"], dtype=torch.float64, device="cuda")
    if kind == "refine":
        # tolerances of the benchmark's precision form
        opts = gsr.solve_opts(itnlim=2000, fixed_iters=False, atol=1e-10, btol=1e-10,
                              precision=gsr.GSR_F32V, max_refine=4, refine_tol=1e-9,
                              refine_first_tol=1e-6)
        return dict(case=case, h=_open(s, build_f32=True), b=b, x=x, opts=opts)
    if kind == "con":
        con, c = _constraints(case, s, gen)
        h = _open(s)
        gsr.gsr_set_constraints(h, *con)
        return dict(case=case, h=h, b=torch.cat([b, c]), x=x,
                    opts=gsr.solve_opts(itnlim=2000, fixed_iters=False, atol=1e-12, btol=1e-12))
    return dict(case=case, h=_open(s), b=b, x=x, var=torch.empty_like(x),
                opts=gsr.solve_opts(itnlim=case["iters"], fixed_iters=True))


def run(state):
    kind = state["case"]["kind"]
    if kind == "products":
        f32 = state["case"]["f32"]
        state["ax"].zero_()
        (gsr.gsr_aprod1_f32v if f32 else gsr.gsr_aprod1)(state["h"], state["x"], state["ax"])
        state["aty"].zero_()
        (gsr.gsr_aprod2_f32v if f32 else gsr.gsr_aprod2)(state["h"], state["y"], state["aty"])
        return state["ax"], state["aty"]
    if kind == "grad":
        x = autograd.lstsq(state["vals"], state["b"], state["structure"], itnlim=2000, atol=1e-12,
                           btol=1e-12)
        loss = 0.5 * (x - state["x_ref"]).square().sum()
        gv, gb = torch.autograd.grad(loss, (state["vals"], state["b"]))
        return x.detach(), gv, gb
    if kind == "batch":
        gsr.gsr_batch_solve(state["b"], state["rhs"], state["x"], state["opts"])
        return state["x"]
    if state["case"].get("var"):
        gsr.gsr_lsqr_solve_var(state["h"], state["b"], state["x"], state["var"], state["opts"])
        return state["x"], state["var"]
    gsr.gsr_lsqr_solve(state["h"], state["b"], state["x"], state["opts"])
    return state["x"]


# ---- what a pass cannot do without --------------------------------------------------------

def _sizes(case):
    m = case["stars"] * 0.5 * (case["obs_lo"] + case["obs_hi"])
    return m, 5 * case["stars"] + 3 * case["n_dfa"] + case["n_instr"] + 1


def _solve_work(m, n, iters, coef=8, k=1):
    """PC-LSQR: every iteration reads each row's coefficients and indices once, u (read and
    write), and v, w, z (read and write) and p; the initial product reads the rows once more.
    Per iteration 2 products of 24 terms a row and about 10 operations an unknown."""
    return dict(bytes=(iters + 1) * (m * (24 * coef + 32 + 16 * k) + n * (48 * k + 8)),
                flops=k * ((2 * iters + 1) * 48.0 * m + iters * 10.0 * n))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        stars = _batch_stars(case)
        iters = case["iters"] if case["tol"] == 0.0 else 60
        m = sum(35.0 * s for s in stars)
        n = sum(5 * s + 3 * max(4, s // 10) + case["n_instr"] + 1 for s in stars)
        return _solve_work(m, n, iters, k=case["k"])
    m, n = _sizes(case)
    if kind == "products":
        # each product reads the rows and one vector and writes the other
        coef = 4 if case["f32"] else 8
        return dict(bytes=2 * (m * (24 * coef + 32 + 8) + 8 * n), flops=2 * 48.0 * m)
    if kind == "grad":
        # forward solve, adjoint solve and the second solve of the backward pass, about 70
        # iterations each, and the coefficient gradient
        w = _solve_work(m, n, 210)
        return dict(bytes=w["bytes"] + m * (192 + 32 + 16 + 192) + 16 * n,
                    flops=w["flops"] + 3 * 24.0 * m)
    if kind == "refine":
        return _solve_work(m, n, 95, coef=4)
    w = _solve_work(m, n, 80 if kind == "con" else case["iters"])
    if case.get("var"):
        w["bytes"] += case["iters"] * 16 * n
    return w


# ---- the same in plain torch, binary64 -----------------------------------------------------

def _cols(s, r0, r1):
    """Columns of the 24 coefficients of rows r0..r1."""
    if "cols" in s:
        return s["cols"][r0:r1]
    d = "cuda"
    a = torch.arange(5, device=d)
    j = torch.arange(4, device=d)
    base = 5 * s["stars"]
    star = s["star"][r0:r1].to(torch.int64)[:, None]
    att = s["att"][r0:r1].to(torch.int64)[:, None]
    ins = s["instr"][6 * r0:6 * r1].to(torch.int64).reshape(-1, 6)
    parts = [5 * star + a] + [base + ax * s["n_dfa"] + att + j for ax in range(3)]
    parts.append(base + 3 * s["n_dfa"] + ins)
    parts.append(torch.full_like(star, s["n"] - 1))
    return torch.cat(parts, 1)


def _coefs(s, r0, r1):
    v = s["vals"].detach()[24 * r0:24 * r1].reshape(-1, 24)
    return v.to(torch.float32).to(torch.float64) if s.get("round32") else v


def _times(s, x):
    """A x (x [n] or [n, k])."""
    out = []
    for r0 in range(0, s["m"], CHUNK):
        r1 = min(s["m"], r0 + CHUNK)
        c, v = _cols(s, r0, r1), _coefs(s, r0, r1)
        y = torch.zeros((r1 - r0,) + tuple(x.shape[1:]), dtype=torch.float64, device="cuda")
        for k in range(24):
            vk = v[:, k] if x.dim() == 1 else v[:, k:k + 1]
            y += vk * x[c[:, k]]
        out.append(y)
    if "con" in s:
        ptr, col, val = s["con"]
        out.append(torch.stack([(val[a:b] * x[col[a:b]]).sum()
                                for a, b in zip(ptr.tolist()[:-1], ptr.tolist()[1:])]))
    return torch.cat(out)


def _scatter(s, weights, square=False):
    """sum_i A[i, c] y_i (y = weights) or, with `square`, sum_i A[i, c]^2, per column c: the
    columns that many rows share are summed into a few copies first, which keeps the adds to
    one address apart; a star's rows are contiguous and summed as a segment."""
    tail = tuple(weights.shape[1:]) if weights is not None else ()
    one = 0 if "cols" in s else 5 * s["stars"]  # columns before it go by segments
    copies = 32
    x = torch.zeros((copies, s["n"] - one) + tail, dtype=torch.float64, device="cuda")
    flat = x.reshape((-1,) + tail)
    glob = 0.0
    head = []
    for r0 in range(0, s["m"], CHUNK):
        r1 = min(s["m"], r0 + CHUNK)
        c, v = _cols(s, r0, r1), _coefs(s, r0, r1)
        copy = (torch.arange(r1 - r0, device="cuda") % copies) * (s["n"] - one) - one

        def term(k, v=v, r0=r0, r1=r1):
            if square:
                return v[:, k].square()
            return v[:, k] * weights[r0:r1] if not tail else v[:, k:k + 1] * weights[r0:r1]

        for k in range(0 if "cols" in s else 5, 24):
            if k == 23 and "cols" not in s:
                glob = glob + term(k).sum(0)
            else:
                flat.index_add_(0, c[:, k] + copy, term(k))
        if "cols" not in s:
            stars, counts = torch.unique_consecutive(s["star"][r0:r1], return_counts=True)
            data = torch.stack([term(k) for k in range(5)], 1)
            head.append((stars.to(torch.int64), torch.segment_reduce(data, "sum", lengths=counts,
                                                                     axis=0)))
    out = x.sum(0)
    if "cols" in s:
        return out
    out[-1] += glob
    astro = torch.zeros((s["stars"], 5) + tail, dtype=torch.float64, device="cuda")
    for stars, sums in head:
        astro.index_add_(0, stars, sums)
    return torch.cat([astro.reshape((-1,) + tail), out])


def _trans(s, y):
    """A^T y."""
    x = _scatter(s, y)
    if "con" in s:
        ptr, col, val = s["con"]
        p = ptr.tolist()
        for k, (a, b) in enumerate(zip(p[:-1], p[1:])):
            x.index_add_(0, col[a:b], val[a:b] * y[s["m"] + k])
    return x


def _precond(s):
    ss = _scatter(s, None, square=True)
    if "con" in s:
        ss.index_add_(0, s["con"][1], s["con"][2].square())
    return torch.where(ss > 0, ss.rsqrt(), torch.zeros_like(ss))


def _lsqr(s, b, iters):
    """Paige & Saunders' LSQR on A D, D = diag(1 / column norms), a fixed number of steps:
    x = D z and the running sum of (D w_i / rho_i)^2."""
    p = _precond(s)
    pd = p if b.dim() == 1 else p[:, None]
    norm = lambda t: t.square().sum(0).sqrt()  # noqa: E731
    beta = norm(b)
    u = b / beta
    v = pd * _trans(s, u)
    alpha = norm(v)
    v = v / alpha
    w, z, var = v.clone(), torch.zeros_like(v), torch.zeros_like(v)
    rhobar, phibar = alpha, beta
    for _ in range(iters):
        u = _times(s, pd * v) - alpha * u
        beta = norm(u)
        u = u / beta
        v = pd * _trans(s, u) - beta * v
        alpha = norm(v)
        v = v / alpha
        rho = torch.sqrt(rhobar * rhobar + beta * beta)
        c, sn = rhobar / rho, beta / rho
        z = z + (c * phibar / rho) * w
        var = var + (w / rho).square()
        w = v - (sn * alpha / rho) * w
        rhobar, phibar = -c * alpha, sn * phibar
    return pd * z, pd * pd * var


def _together(systems):
    """Several systems as one block-diagonal system with its columns written out."""
    cols, n = [], 0
    for s in systems:
        cols.append(_cols(s, 0, s["m"]) + n)
        n += s["n"]
    return dict(m=sum(s["m"] for s in systems), n=n, cols=torch.cat(cols),
                vals=torch.cat([s["vals"] for s in systems]))


def _normal_solve(s, g, drop=1e-15, steps=200):
    """(A^T A)^-1 g by conjugate gradients on the column-scaled normal equations, until the
    residual has fallen by the factor `drop`."""
    p = _precond(s)
    pd = p if g.dim() == 1 else p[:, None]
    r = pd * g
    x = torch.zeros_like(r)
    d, rr = r.clone(), r.square().sum(0)
    first = rr.clone()
    for _ in range(steps):
        q = pd * _trans(s, _times(s, pd * d))
        a = rr / (d * q).sum(0)
        a = torch.where(rr > 0, a, torch.zeros_like(a))
        x = x + a * d
        r = r - a * q
        new = r.square().sum(0)
        d = r + torch.where(rr > 0, new / rr, torch.zeros_like(rr)) * d
        rr = new
        if bool((rr <= drop * drop * first).all()):
            break
    return pd * x


def _lstsq(s, b):
    x = _normal_solve(s, _trans(s, b))
    return x + _normal_solve(s, _trans(s, b - _times(s, x)), 1e-4)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        systems = _batch_systems(case, seed)
        if case["tol"] == 0.0:
            return torch.cat([_lsqr(s, b, case["iters"])[0].reshape(-1) for s, b in systems])
        return _lstsq(_together([s for s, _ in systems]), torch.cat([b for _, b in systems])).reshape(-1)
    s, gen = _one_system(case, seed)
    if kind == "products":
        s["round32"] = case["f32"]
        x, y = _normal(s["n"], gen), _normal(s["m"], gen)
        return _times(s, x), _trans(s, y)
    b = _rhs(s, gen)
    if kind == "grad":
        x_ref = _normal(s["n"], gen)
        x = _lstsq(s, b)
        g = x - x_ref
        lam = _normal_solve(s, g)
        mu, r = _times(s, lam), b - _times(s, x)
        gv = torch.cat([(r[r0:r0 + CHUNK, None] * lam[c] - mu[r0:r0 + CHUNK, None] * x[c]).reshape(-1)
                        for r0 in range(0, s["m"], CHUNK)
                        for c in (_cols(s, r0, min(s["m"], r0 + CHUNK)),)])
        return x, gv, mu
    if kind == "refine":
        return _lstsq(s, b)
    if kind == "con":
        s["con"], c = _constraints(case, s, gen)
        return _lstsq(s, torch.cat([b, c]))
    x, var = _lsqr(s, b, case["iters"])
    return (x, var) if case.get("var") else x

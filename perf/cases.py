"""Performance cases of the RGDBEK solver: what a program asks of it, through
the package's public entry points.

Each case names a kind of use and its sizes.  Inputs are made on the GPU from
the seed alone; `prepare` also makes the solver handle where a program keeps
one (many right-hand sides one after the other, iterations of a larger
method), and `run` makes it where a program has a new matrix on every call.
"""
import math

import numpy as np
import torch

import paper_2509_19267_amd as rg

F64 = torch.float64


def listed():
    return [
        # one block draw on given weights, at the row count of the dense
        # least-squares workload: the smallest call, all latency
        dict(name="draw_20000_k4000", kind="draw", d=20000, k=4000),
        # the residual products A x and A^T z of a power-law matrix, alone
        # (the sparse workload's SpMV figures), FP64 and FP32 storage
        dict(name="apply_powerlaw_1m_f64", kind="apply", m=1000000, n=500000,
             form="f64"),
        dict(name="apply_powerlaw_300k_f32", kind="apply", m=300001, n=150001,
             form="f32"),
        # the small dense consistent system, solved to 1e-8: a hundred
        # iterations of small blocks, bound by launches and serial chains
        dict(name="consistent_500x250", kind="consistent", m=500, n=250,
             eta=0.5, tol=1e-8),
        # a differentiable layer whose matrix changes at every step: set-up,
        # forward, and the gradients in A and b, at odd sizes
        dict(name="layer_2003x501", kind="layer", m=2003, n=501, k_col=301,
             k_row=301, tol=1e-10),
        # the dense least-squares workload at its tuned settings, plain FP64
        # and FP32 iterations inside FP64 refinement
        dict(name="lsq_20000x5000_fp64", kind="lsq", m=20000, n=5000,
             k_col=4000, k_row=4000, form="fp64", inner_tol=0.03, inner_max=8,
             tile_rows=400, tol=1e-8),
        dict(name="lsq_20000x5000_mixed", kind="lsq", m=20000, n=5000,
             k_col=4500, k_row=4500, form="mixed_f32", inner_tol=0.1,
             inner_max=16, tile_rows=224, tol=1e-10),
        # the random sparse comparison of the paper's Section 3 (row blocks
        # taller than the matrix is wide), to its squared residual test
        dict(name="sparse_8000x500_rse", kind="uniform", m=8000, n=500,
             eta=0.5, stop="rse", tol=1e-6, iters=30),
        # a small sparse system with exact projections, through its Grams
        dict(name="sparse_3000x1500", kind="uniform", m=3000, n=1500,
             eta=0.25, stop="none", tol=0.0, iters=10),
        # iterations of the large power-law system at its tuned settings
        dict(name="powerlaw_1m_fp64", kind="powerlaw", m=1000000, n=500000,
             eta=0.5, iters=16),
        # a batch of uneven grid systems solved together, FP32 storage and
        # FP64 refinement
        dict(name="grids_12_mixed", kind="grids", count=12, n_min=2000,
             n_max=20000, form="mixed_f32", eta=0.7, tol=1e-10),
        # deblurring of 64 images at once with Tikhonov rows, FP32 storage
        # and FP64 refinement
        dict(name="deblur_256_rhs64_mixed", kind="deblur", npix=256, nrhs=64,
             form="mixed_f32", eta=0.5, tol=1e-11, iters=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["draw", "apply", "consistent", "layer", "lsq", "lsq",
                       "uniform", "uniform", "powerlaw", "grids", "deblur"])
    if kind == "draw":
        d = _log(rng, 500, 1000000)
        return dict(kind=kind, d=d, k=max(1, int(d * rng.uniform(0.05, 0.5))))
    if kind == "apply":
        m = _log(rng, 20000, 1000000)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(0.3, 0.9)),
                    form=rng.choice(["f64", "f32"]))
    if kind == "consistent":
        m = _log(rng, 150, 900)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(0.4, 0.55)),
                    eta=round(rng.uniform(0.2, 0.4), 3), tol=1e-8)
    if kind == "layer":
        m = _log(rng, 800, 4000)
        n = int(m * rng.uniform(0.2, 0.3))
        k = int(n * rng.uniform(0.3, 0.65))
        return dict(kind=kind, m=m, n=n, k_col=k, k_row=k, tol=1e-10)
    if kind == "lsq":
        m = _log(rng, 4000, 20000)
        n = int(m * rng.uniform(0.2, 0.25))
        k = int(n * rng.uniform(0.5, 0.8))
        if rng.random() < 0.5:
            return dict(kind=kind, m=m, n=n, k_col=k, k_row=k, form="fp64",
                        inner_tol=0.03, inner_max=8, tile_rows=0, tol=1e-8)
        return dict(kind=kind, m=m, n=n, k_col=k, k_row=k, form="mixed_f32",
                    inner_tol=0.1, inner_max=16, tile_rows=0, tol=1e-10)
    if kind == "uniform":
        if rng.random() < 0.5:
            return dict(kind=kind, m=rng.randint(4200, 9000),
                        n=rng.randint(300, 900), eta=0.5, stop="rse",
                        tol=1e-6, iters=30)
        m = rng.randint(1500, 4000)
        return dict(kind=kind, m=m, n=m // 2 - rng.randint(0, 99),
                    eta=round(rng.uniform(0.1, 0.25), 3), stop="none",
                    tol=0.0, iters=10)
    if kind == "powerlaw":
        m = _log(rng, 60000, 1000000)
        return dict(kind=kind, m=m, n=int(m * rng.uniform(0.4, 0.6)),
                    eta=round(rng.uniform(0.1, 0.5), 3),
                    iters=rng.randint(8, 16))
    if kind == "grids":
        return dict(kind=kind, count=rng.randint(4, 12), n_min=2000,
                    n_max=_log(rng, 4000, 20000),
                    form=rng.choice(["fp64", "mixed_f32"]), eta=0.7,
                    tol=1e-10)
    npix = rng.randint(96, 200)
    return dict(kind="deblur", npix=npix, nrhs=rng.choice([4, 16, 20, 32, 64]),
                form="fp64", eta=0.5, tol=0.0, iters=rng.randint(4, 8))


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=F64, device="cuda")


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=F64, device="cuda")


def _row_sums(v, rp):
    return torch.segment_reduce(v, "sum", offsets=rp)


def _csr_product(csr, x):
    rp, ci, v = csr
    return _row_sums(v.double() * x[ci.long()], rp)


def _csr_from_keys(keys, m, n):
    """Row pointers and column indices of the distinct sorted row*n + col."""
    rows = torch.div(keys, n, rounding_mode="floor")
    rp = torch.searchsorted(rows, torch.arange(m + 1, device="cuda"))
    return rp, (keys - rows * n).to(torch.int32)


def _powerlaw(case, seed):
    """Row lengths 1..2000 from a power law of mean 10, uniform columns,
    N(0,1) values, rows of unit norm; b = A x*."""
    m, n = case["m"], case["n"]
    g = _gen(seed)
    ls = np.arange(1, 2001, dtype=np.float64)
    lo, hi = 0.0, 10.0
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        w = ls ** -mid
        lo, hi = (mid, hi) if (ls * w).sum() / w.sum() > 10.0 else (lo, mid)
    cdf = torch.as_tensor(np.cumsum(w / w.sum())).cuda()
    lens = torch.searchsorted(cdf, _rand(g, m)).clamp_(max=1999) + 1
    rows = torch.repeat_interleave(torch.arange(m, device="cuda"), lens)
    cols = torch.randint(0, n, rows.shape, generator=g, device="cuda")
    rp, ci = _csr_from_keys(torch.unique(rows * n + cols), m, n)
    v = _randn(g, ci.numel())
    norm = _row_sums(v * v, rp).sqrt()
    v = v / torch.repeat_interleave(norm, rp[1:] - rp[:-1])
    csr = (rp, ci, v)
    x = _randn(g, n)
    return csr, _csr_product(csr, x), x, g


def _uniform(case, seed):
    """1% of the positions at random, N(0,1) values; b = A x*."""
    m, n = case["m"], case["n"]
    g = _gen(seed)
    keys = torch.unique(torch.randint(0, m * n, (m * n // 100,), generator=g,
                                      device="cuda"))
    rp, ci = _csr_from_keys(keys, m, n)
    csr = (rp, ci, _randn(g, ci.numel()))
    x = _randn(g, n)
    return csr, _csr_product(csr, x), x


def _dense(case, seed):
    """N(0,1) entries, x* ~ N(0,1); least squares: b = A x* + r with r in
    null(A^T), ||r|| = 0.1 ||A x*||."""
    m, n = case["m"], case["n"]
    g = _gen(seed)
    a, x = _randn(g, m, n), _randn(g, n)
    b = a @ x
    if case["kind"] == "consistent":
        return a, b, x, None
    r = _randn(g, m)
    ch = torch.linalg.cholesky(a.t() @ a)
    for _ in range(2):
        r = r - a @ torch.cholesky_solve((a.t() @ r)[:, None], ch)[:, 0]
    r *= 0.1 * b.norm() / r.norm()
    return a, b + r, x, r


def _grids(case, seed):
    """Shifted 5-point Laplacians on uneven grids, a fifth more rows of 8
    random entries each, block-diagonal; FP32 values, b = A x* in FP64."""
    g = _gen(seed)
    sizes = np.random.default_rng([case["count"], case["n_min"], case["n_max"]])
    ro, co, keys, vals = [0], [0], [], []
    grids = []
    for _ in range(case["count"]):
        ns = math.exp(sizes.uniform(math.log(case["n_min"]),
                                    math.log(case["n_max"])))
        nx = max(2, round(math.sqrt(ns)))
        ny = max(2, round(ns / nx))
        grids.append((nx, ny, sizes.uniform(0.1, 1.0)))
    n = sum(nx * ny for nx, ny, _ in grids)
    for nx, ny, shift in grids:
        ns = nx * ny
        i = torch.arange(ns, device="cuda")
        px, py = i % nx, torch.div(i, nx, rounding_mode="floor")
        for off, ok, v in ((0, px >= 0, 4.0 + shift), (-1, px > 0, -1.0),
                           (1, px < nx - 1, -1.0), (-nx, py > 0, -1.0),
                           (nx, py < ny - 1, -1.0)):
            r = i[ok]
            keys.append((ro[-1] + r) * n + co[-1] + r + off)
            vals.append(torch.full((r.numel(),), v, dtype=F64, device="cuda"))
        ne = round(0.2 * ns)
        r = torch.arange(ne, device="cuda").repeat_interleave(8)
        c = torch.randint(0, ns, r.shape, generator=g, device="cuda")
        k = torch.unique((ro[-1] + ns + r) * n + co[-1] + c)
        keys.append(k)
        vals.append(_randn(g, k.numel()))
        ro.append(ro[-1] + ns + ne)
        co.append(co[-1] + ns)
    keys, order = torch.sort(torch.cat(keys))
    rp, ci = _csr_from_keys(keys, ro[-1], n)
    csr = (rp, ci, torch.cat(vals)[order].float())
    x = _randn(g, n)
    return csr, ro, co, _csr_product(csr, x), x


def _psf():
    d = np.arange(-7, 8, dtype=np.float64)
    w = np.exp(-d * d / 8.0) / (2.0 * math.sqrt(2.0 * math.pi))
    f, e = np.frexp(w)   # 12 bits: products of two are exact in FP32
    return np.ldexp(np.round(f * 4096.0) / 4096.0, e)


S = float(np.float32(0.1))   # Tikhonov weight


def _deblur(case, seed):
    """[A; s I] with A the separable Gaussian blur (sigma 2, 15 x 15, zero
    boundary), s^2 = 0.01; blurred smooth fields with 1% noise."""
    p, nrhs = case["npix"], case["nrhs"]
    n = p * p
    g = _gen(seed)
    w = torch.as_tensor(_psf()).cuda()
    i = torch.arange(n, device="cuda")
    off = torch.arange(-7, 8, device="cuda")
    y = torch.div(i, p, rounding_mode="floor")[:, None] + off
    x = (i % p)[:, None] + off
    ok = (((y >= 0) & (y < p))[:, :, None] & ((x >= 0) & (x < p))[:, None, :])
    ci = (y[:, :, None] * p + x[:, None, :])[ok]
    v = (w[:, None] * w[None, :]).expand(n, 15, 15)[ok]
    lens = ok.sum(dim=(1, 2))
    rp = torch.zeros(2 * n + 1, dtype=torch.int64, device="cuda")
    rp[1:n + 1] = torch.cumsum(lens, 0)
    rp[n + 1:] = rp[n] + i + 1
    csr = (rp, torch.cat([ci, i]).to(torch.int32),
           torch.cat([v, torch.full((n,), S, dtype=F64, device="cuda")]).float())
    t = torch.zeros(p, p, dtype=F64, device="cuda")
    for o in range(-7, 8):
        t += torch.diag(w[o + 7].expand(p - abs(o)), o)
    f = torch.fft.fftfreq(p, dtype=F64, device="cuda")
    filt = torch.exp(-2.0 * (math.pi * 8.0) ** 2 * (f[:, None] ** 2 + f[None, :] ** 2))
    img = torch.fft.ifft2(torch.fft.fft2(_randn(g, nrhs, p, p)) * filt).real
    img = (img - img.mean(dim=(1, 2), keepdim=True)) / img.std(dim=(1, 2), keepdim=True)
    img = t @ img.reshape(nrhs * p, p).t().reshape(p, nrhs * p)   # T X, columns
    img = img.reshape(p, nrhs, p).permute(1, 2, 0).reshape(nrhs * p, p) @ t
    img = img.reshape(nrhs, p, p)
    img = img + 0.01 * img.std(dim=(1, 2), keepdim=True) * _randn(g, nrhs, p, p)
    b = torch.zeros(nrhs, 2 * n, dtype=F64, device="cuda")
    b[:, :n] = img.reshape(nrhs, n)
    return csr, t, b


# ---------------------------------------------------------------- cases
def prepare(case, seed):
    kind = case["kind"]
    if kind == "draw":
        # residual weights: squares of residual entries over squared norms
        g = _gen(seed)
        return dict(case=case, it=0, eps=_randn(g, case["d"]) ** 2 /
                    (1.0 + _rand(g, case["d"])))
    if kind == "apply":
        csr, _, x, g = _powerlaw(case, seed)
        f32 = case["form"] == "f32"
        s = rg.Solver(csr=csr, shape=(case["m"], case["n"]), eta=0.1,
                      precision="mixed_f32" if f32 else "fp64")
        z = _randn(g, case["m"])
        return dict(case=case, s=s, x=x.float() if f32 else x,
                    z=z.float() if f32 else z)
    if kind in ("consistent", "lsq"):
        a, b, x, _ = _dense(case, seed)
        if kind == "consistent":
            s = rg.Solver(a, eta=case["eta"], stop="err_ref", tol=case["tol"],
                          max_iter=2000)
        else:
            s = rg.Solver(a, k_col=case["k_col"], k_row=case["k_row"],
                          stop="err_ref", tol=case["tol"],
                          precision=case["form"],
                          inner_tol=case["inner_tol"],
                          inner_max=case["inner_max"],
                          tile_rows=case["tile_rows"], gram_aat=True,
                          pass_drop=1e-4 if case["form"] == "mixed_f32" else 0.0)
        return dict(case=case, s=s, b=b, x=x)
    if kind == "layer":
        a, b, _, _ = _dense(case, seed)
        c = _randn(_gen(seed + 1), case["n"])
        return dict(case=case, a=a, b=b, c=c)
    if kind == "uniform":
        csr, b, _ = _uniform(case, seed)
        s = rg.Solver(csr=csr, shape=(case["m"], case["n"]), eta=case["eta"],
                      stop=case["stop"], tol=case["tol"],
                      max_iter=case["iters"])
        return dict(case=case, s=s, b=b)
    if kind == "powerlaw":
        csr, b, _, _ = _powerlaw(case, seed)
        s = rg.Solver(csr=csr, shape=(case["m"], case["n"]), eta=case["eta"],
                      stop="none", max_iter=case["iters"], inner_tol=0.1,
                      inner_max=8)
        return dict(case=case, s=s, b=b)
    if kind == "grids":
        csr, ro, co, b, x = _grids(case, seed)
        s = rg.BatchSolver(csr, ro, co, eta=case["eta"], stop="err_ref",
                           tol=case["tol"], precision=case["form"],
                           inner_tol=0.1, inner_max=8,
                           pass_drop=1e-3 if case["form"] == "mixed_f32" else 0.0)
        return dict(case=case, s=s, b=b, x=x)
    csr, _, b = _deblur(case, seed)
    n = case["npix"] ** 2
    s = rg.MultiRhsSolver(csr, (2 * n, n), case["nrhs"], eta=case["eta"],
                          stop="none" if case["iters"] else "res_ext",
                          tol=case["tol"], max_iter=case["iters"] or 2000,
                          precision=case["form"], inner_tol=0.1, inner_max=8,
                          graph_iters=4)
    return dict(case=case, s=s, b=b.reshape(-1))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "draw":
        return rg.select(state["eps"], case["k"], seed=1, it=3, phase=1)
    s = state.get("s")
    if kind == "apply":
        return s.apply(state["x"], state["z"], precision=case["form"])
    if kind == "layer":
        values = state["a"].reshape(-1).detach().requires_grad_(True)
        b = state["b"].detach().requires_grad_(True)
        with rg.Solver(state["a"], k_col=case["k_col"], k_row=case["k_row"],
                       stop="res_ext", tol=case["tol"]) as s:
            x = rg.solve(s, values, b, least_squares=True)
            da, db = torch.autograd.grad((x * state["c"]).sum(), (values, b))
        return x.detach(), da, db
    x, _ = s.solve(state["b"], state.get("x"))
    if not _returns_z(case):
        return x
    return x, s.get_z()


def _returns_z(case):
    """Whether a program keeps z: the least-squares residual, or the state of
    a run that goes on.  (On consistent systems it only tends to zero; the
    mixed form's is the last pass's estimate.)"""
    if case.get("form") == "mixed_f32" or case["kind"] in ("consistent", "grids"):
        return False
    return case.get("stop") != "rse"


def work(case):
    """Bytes read and written once and operations per pass.  A solve reads
    all of A once per iteration for both residuals and its column and row
    blocks once for the updates; iteration counts are those of the listed
    sizes where a solve runs to a tolerance."""
    kind = case["kind"]
    if kind == "draw":
        return dict(bytes=8.0 * case["d"] + 4.0 * case["k"],
                    flops=20.0 * case["d"])
    m, n = case.get("m"), case.get("n")
    if kind in ("apply", "powerlaw"):
        v = 4.0 if case.get("form") == "f32" else 8.0
        nnz = 10.0 * m
        one = 2 * nnz * (v + 4) + 8 * (m + n) + 2 * v * (m + n)
        if kind == "apply":
            return dict(bytes=one, flops=4 * nnz)
        its = case["iters"]
        return dict(bytes=its * one * (1 + case["eta"]),
                    flops=its * 4 * nnz * (1 + case["eta"]))
    if kind in ("consistent", "lsq", "layer"):
        kc = case.get("k_col") or case["eta"] * n
        kr = case.get("k_row") or case["eta"] * m
        f32 = case.get("form") == "mixed_f32"
        its = {"consistent": 90, "lsq": 27 if f32 else 21, "layer": 100}[kind]
        el = its * (m * n + kc * m + kr * n)
        return dict(bytes=(4.0 if f32 else 8.0) * el, flops=2.0 * el)
    if kind == "uniform":
        its = 6 if case["stop"] == "rse" else case["iters"]
        nnz = 0.01 * m * n
        return dict(bytes=its * 2 * nnz * 12.0 * (1 + case["eta"]),
                    flops=its * 4 * nnz * (1 + case["eta"]))
    if kind == "grids":
        mean = (case["n_max"] - case["n_min"]) / math.log(case["n_max"] / case["n_min"])
        nnz = 6.6 * mean * case["count"]
        v = 4.0 if case["form"] == "mixed_f32" else 8.0
        return dict(bytes=200 * 2 * nnz * (v + 4) * (1 + case["eta"]),
                    flops=200 * 4 * nnz * (1 + case["eta"]))
    n = case["npix"] ** 2
    nnz, its = 226.0 * n, case["iters"] or 50
    v = 4.0 if case["form"] == "mixed_f32" else 8.0
    return dict(bytes=its * (2 * nnz * (v + 4) + case["nrhs"] * 8 * n * v),
                flops=its * 4 * nnz * case["nrhs"] * (1 + case["eta"]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "draw" or kind == "powerlaw":
        return None
    if kind == "apply":
        (rp, ci, v), _, x, g = _powerlaw(case, seed)
        z = _randn(g, case["m"])
        if case["form"] == "f32":
            x, z, v = x.float().double(), z.float().double(), v.float().double()
        rows = torch.repeat_interleave(torch.arange(case["m"], device="cuda"),
                                       rp[1:] - rp[:-1])
        atz = torch.zeros(case["n"], dtype=F64, device="cuda")
        atz.index_add_(0, ci.long(), v * z[rows])
        return _csr_product((rp, ci, v), x), atz
    if kind == "consistent":
        return _dense(case, seed)[2]
    if kind == "lsq":
        _, _, x, r = _dense(case, seed)
        return x if case["form"] == "mixed_f32" else (x, r)
    if kind == "layer":
        a, b, _, _ = _dense(case, seed)
        c = _randn(_gen(seed + 1), case["n"])
        q, up = torch.linalg.qr(a)

        def pinv(v):
            return torch.linalg.solve_triangular(up, (q.t() @ v)[:, None],
                                                 upper=True)[:, 0]
        x = pinv(b)
        w = q @ torch.linalg.solve_triangular(up.t(), c[:, None], upper=False)[:, 0]
        da = torch.outer(b - a @ x, pinv(w)) - torch.outer(w, x)
        return x, da.reshape(-1), w
    if kind == "uniform":
        if case["stop"] == "none":
            return None
        return _uniform(case, seed)[2]
    if kind == "grids":
        return _grids(case, seed)[4]
    if case["iters"]:
        return None
    _, t, b = _deblur(case, seed)
    p, nrhs = case["npix"], case["nrhs"]
    lam, q = torch.linalg.eigh(t)
    y = b[:, :p * p].reshape(nrhs, p, p)
    two = lam[:, None] * lam[None, :]
    c = torch.stack([q.t() @ u @ q for u in y]) * (two / (two * two + S * S))
    return torch.stack([q @ u @ q.t() for u in c]).reshape(-1)

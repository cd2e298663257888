"""Launches whose workgroups exchange values, with fewer workgroups than the
launch has (as when another stream's launch holds part of the device): the
others take over their shares and the results are the same bit for bit.  The
size is capped from the host; the workgroups above it leave as late ones do."""
import ctypes
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _limit(s, n):
    f = s._lib.rgdbek_debug_team_limit
    f.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    assert f(s._h, n) == 0


def _sparse(m, n, per_row, seed):
    rng = np.random.default_rng(seed)
    keys = np.unique(rng.integers(0, m * n, m * per_row))
    r = keys // n
    rp = np.searchsorted(r, np.arange(m + 1))
    v = rng.standard_normal(len(keys))
    v /= np.sqrt(np.maximum(1e-300, np.bincount(r, v * v, m)))[r]
    x = rng.standard_normal(n)
    b = np.bincount(r, v * x[keys % n], m) + 0.1 * rng.standard_normal(m)
    return (torch.as_tensor(rp.astype(np.int64)).cuda(),
            torch.as_tensor((keys % n).astype(np.int32)).cuda(),
            torch.as_tensor(v).cuda()), torch.as_tensor(b).cuda()


def _solves(s, b, limits):
    out = []
    for n in limits:
        _limit(s, n)
        x, _ = s.solve(b)
        out.append((x, s.get_z()))
        print("team", n, flush=True)
    s.close()
    for x, z in out[1:]:
        assert torch.equal(x, out[0][0]) and torch.equal(z, out[0][1])


# columns and rows, of one and of more segments per lane group; tall row blocks
@pytest.mark.parametrize("m,n,per_row,kc,kr", [
    (700, 900, 40, 300, 350), (9000, 6000, 5, 4000, 5000),
    (60000, 30000, 6, 20000, 26000), (2600, 60, 20, 30, 1300),
    (9000, 700, 40, 350, 4500), (60000, 300, 2, 150, 30000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed_f32"])
def test_sparse_cg(rg, m, n, per_row, kc, kr, precision):
    csr, b = _sparse(m, n, per_row, m + n)
    s = rg.Solver(csr=csr, shape=(m, n), k_col=kc, k_row=kr, seed=3,
                  stop="none" if precision == "fp64" else "res_ext",
                  tol=1e-30, max_iter=3, inner_max=4, inner_tol=1e-14,
                  sparse_cg=True, precision=precision)
    _solves(s, b, [0, 1, 3, 50, 255, 0])


# blocks of one and of several columns per thread; rows kept in registers, in
# LDS and streamed, more of them the smaller the team; gathered from a
# precomputed Gram or formed from the rows
@pytest.mark.parametrize("m,n,k,precision,gram_aat", [
    (900, 700, 300, "fp64", True), (900, 700, 301, "mixed_f32", False),
    (2600, 1700, 1100, "fp64", True), (4000, 2600, 2050, "fp64", False),
    (7000, 4200, 4000, "fp64", True), (7000, 5000, 4500, "mixed_f32", True)])
def test_pcg(rg, m, n, k, precision, gram_aat):
    g = torch.Generator(device="cuda").manual_seed(k)
    a = torch.randn(m, n, generator=g, dtype=torch.float64, device="cuda")
    b = torch.randn(m, generator=g, dtype=torch.float64, device="cuda")
    s = rg.Solver(a, k_col=k, k_row=k, seed=1, max_iter=3, inner_max=9,
                  stop="none" if precision == "fp64" else "res_ext", tol=1e-30,
                  inner_tol=1e-13, gram_aat=gram_aat, precision=precision,
                  solver=rg._binding.SOLVER_CG)
    _solves(s, b, [0, 1, 3, 30, 100, 255, 0])


@pytest.mark.parametrize("k,threads", [(300, 4), (1100, 3), (1900, 2),
                                       (4000, 2)])
def test_pcg_on_streams(rg, k, threads):
    """Solves at the same time on streams of their own, whose workgroups do
    not all fit the device together: the bits of the solves alone."""
    g = torch.Generator(device="cuda").manual_seed(k)
    a = torch.randn(2 * k, k + 200, generator=g, dtype=torch.float64,
                    device="cuda")
    bs, ss, sts = [], [], []
    for i in range(threads):
        st = torch.cuda.Stream()
        torch.cuda.synchronize()
        sts.append(st)
        bs.append(torch.randn(2 * k, generator=g, dtype=torch.float64,
                              device="cuda"))
        ss.append(rg.Solver(a, k_col=k, k_row=k, stop="none", max_iter=8,
                            seed=i, inner_max=9, stream=st, gram_aat=True,
                            solver=rg._binding.SOLVER_CG))
    torch.cuda.synchronize()

    def solve(i, out):
        try:
            with torch.cuda.stream(sts[i]):
                for _ in range(3):
                    x, _ = ss[i].solve(bs[i])
                sts[i].synchronize()
            out[i] = x
        except Exception as e:       # shown by the thread that compares
            out[i] = e

    alone, both = {}, {}
    for i in range(threads):
        solve(i, alone)
    ts = [threading.Thread(target=solve, args=(i, both)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in range(threads):
        for out in (alone, both):
            if isinstance(out[i], Exception):
                raise out[i]
        assert torch.equal(alone[i], both[i])
        ss[i].close()

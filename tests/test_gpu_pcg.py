"""The persistent block solver at the edges of its layouts: columns per thread
(512, 1024, 2048, 3072, 4096 FP64; up to 8192 FP32), rows kept in registers,
in LDS and streamed, blocks gathered from a precomputed Gram or formed from
the rows.  Reference: the definition of a projection in plain FP64 products
(the block's equations hold after the update), at 1e-10: CG is run to a
residual of 1e-14 and the Grams here have condition numbers below 1e3."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _system(m, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(m, n, generator=g, dtype=torch.float64, device="cuda")
    x = torch.randn(n, generator=g, dtype=torch.float64, device="cuda")
    r = torch.randn(m, generator=g, dtype=torch.float64, device="cuda")
    return a, x, a @ x + r


@pytest.mark.parametrize("k,gram_aat", [
    (257, False), (511, True), (512, True), (513, False), (1025, True),
    (2048, True), (2050, False), (3073, True), (3840, True), (4095, True),
    (4096, False)])
def test_block_equations_hold(rg, k, gram_aat):
    """After one iteration A_U^T z = 0 and A^J x = (b - z)^J."""
    n = max(600, int(1.6 * k))
    m = max(1400, int(1.8 * k))
    a, _, b = _system(m, n, k)
    s = rg.Solver(a, k_col=k, k_row=k, stop="none", max_iter=1, seed=7,
                  inner_max=400, gram_aat=gram_aat, graph_iters=1,
                  solver=rg._binding.SOLVER_CG)
    x, _ = s.solve(b)
    z = s.get_z()
    s.close()
    u = rg.select((a.t() @ b) ** 2 / (a * a).sum(0), k, seed=7).long()
    res = a[:, u].t() @ z
    assert u.numel() == k
    assert res.norm() <= 1e-10 * (a[:, u].t() @ b).norm()
    rhs = b - z
    j = rg.select(rhs ** 2 / (a * a).sum(1), k, seed=7, phase=1).long()
    assert (a[j] @ x - rhs[j]).norm() <= 1e-10 * rhs[j].norm()


@pytest.mark.parametrize("k", [500, 1000, 2000, 4090, 4608, 5200])
def test_mixed_blocks_refine(rg, k):
    """FP32 blocks of every layout refine to the planted solution."""
    n, m = max(1000, k + 300), max(3000, k + 2000)
    a, xs, _ = _system(m, n, k + 1)
    b = a @ xs
    s = rg.Solver(a, k_col=k, k_row=k, stop="err_ref", tol=1e-10,
                  precision="mixed_f32", max_iter=3000, inner_tol=0.05,
                  inner_max=60, gram_aat=True, pass_drop=1e-4)
    x, info = s.solve(b, xs)
    s.close()
    assert info["converged"]
    assert (x - xs).norm() <= 1e-10 * xs.norm()


def test_repeated_launches_and_solves(rg):
    """The exchange buffers rotate over launches of different step counts and
    start every solve empty: solves repeat bit for bit, whatever ran
    before."""
    a, _, b = _system(1500, 700, 3)
    s = rg.Solver(a, k_col=300, k_row=320, stop="none", max_iter=7, seed=1,
                  inner_tol=1e-3, inner_max=9, gram_aat=True,
                  solver=rg._binding.SOLVER_CG)
    x0, _ = s.solve(b)
    s.solve(b * 2 + 1)
    s.solve_adjoint(torch.ones(700, dtype=torch.float64, device="cuda"))
    x1, _ = s.solve(b)
    s.close()
    assert torch.equal(x0, x1)

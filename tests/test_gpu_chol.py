"""The one-workgroup Cholesky block solver at the edges of its 16-column
panels, for consistent and dependent columns.  Reference: the definition of a
projection in plain FP64 products (the block's equations hold after the
update) at 1e-10, the Grams having condition numbers below 1e3."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _matrix(m, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(m, n, generator=g, dtype=torch.float64, device="cuda")
    b = torch.randn(m, generator=g, dtype=torch.float64, device="cuda")
    return a, b


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 33, 113, 128, 250, 256,
                               257, 400, 511, 512])
def test_block_equations_hold(rg, k):
    m, n = max(64, 2 * k), max(40, int(1.7 * k))
    a, b = _matrix(m, n, k)
    s = rg.Solver(a, k_col=k, k_row=k, stop="none", max_iter=1, seed=3,
                  graph_iters=1, solver=rg._binding.SOLVER_CHOL)
    x, _ = s.solve(b)
    z = s.get_z()
    s.close()
    u = rg.select((a.t() @ b) ** 2 / (a * a).sum(0), k, seed=3).long()
    assert (a[:, u].t() @ z).norm() <= 1e-10 * (a[:, u].t() @ b).norm()
    rhs = b - z
    j = rg.select(rhs ** 2 / (a * a).sum(1), k, seed=3, phase=1).long()
    assert (a[j] @ x - rhs[j]).norm() <= 1e-10 * rhs[j].norm()


@pytest.mark.parametrize("n", [40, 90, 250])
def test_dependent_columns(rg, n):
    """A full block with every column twice: the projection is onto the span
    of one copy, the unknowns of the other stay finite."""
    a, b = _matrix(600, n, n)
    a = torch.cat([a, a], dim=1).contiguous()
    s = rg.Solver(a, k_col=2 * n, k_row=1, stop="none", max_iter=1,
                  graph_iters=1, solver=rg._binding.SOLVER_CHOL)
    x, _ = s.solve(b)
    z = s.get_z()
    s.close()
    assert torch.isfinite(x).all()
    assert (a.t() @ z).norm() <= 1e-10 * (a.t() @ b).norm()


@pytest.mark.parametrize("k", [48, 250])
def test_mixed_refines(rg, k):
    a, _ = _matrix(900, 300, k)
    xs = torch.linspace(-1, 1, 300, dtype=torch.float64, device="cuda")
    s = rg.Solver(a, k_col=k, k_row=k, stop="err_ref", tol=1e-10,
                  precision="mixed_f32", max_iter=4000,
                  solver=rg._binding.SOLVER_CHOL)
    x, info = s.solve(a @ xs, xs)
    s.close()
    assert info["converged"]
    assert (x - xs).norm() <= 1e-10 * xs.norm()

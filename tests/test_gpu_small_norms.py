"""Dense mixed solves of matrices whose squared norms are FP32 numbers without
a normal reciprocal.  What limits them there is the residual weights, squares
in FP32: a row with |r_i| < 2^-74.5 has none (2^-149 is the least number), so
the iteration goes on until every row is below that and no further.  Hence
|x - x*| <= 2^-74.5 sqrt(m) / sigma_min, and no numeric error."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("e", [66, 69, 71])
@pytest.mark.parametrize("k,solver,gram_aat", [
    (200, "CHOL", False), (200, "CHOL", True), (400, "CHOL", True),
    (300, "CG", False), (600, "CG", True)])
def test_mixed(e, k, solver, gram_aat):
    import paper_2509_19267_amd as rg
    m, n = 2000, 800
    g = torch.Generator(device="cuda").manual_seed(e + k)
    a = torch.randn(m, n, generator=g, dtype=torch.float64, device="cuda")
    xs = torch.randn(n, generator=g, dtype=torch.float64, device="cuda")
    low = torch.linalg.svdvals(a.cpu())[-1].item() * 2.0 ** -e
    a = a * 2.0 ** -e
    s = rg.Solver(a, k_col=k, k_row=k, stop="err_ref", tol=1e-9, max_iter=3000,
                  precision="mixed_f32", inner_max=60, inner_tol=0.05,
                  solver=getattr(rg._binding, "SOLVER_" + solver),
                  gram_aat=gram_aat)
    x, _ = s.solve(a @ xs, xs)
    s.close()
    err, bound = (x - xs).norm().item(), 2.0 ** -74.5 * m ** 0.5 / low
    print(e, k, solver, err, bound, flush=True)
    assert err <= bound

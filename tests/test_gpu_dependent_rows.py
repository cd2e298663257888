"""Row blocks with every row of a few several times over and right-hand sides
that contradict each other: A A^T is singular and the CG's residual ends in its
null space.  The solve stays finite (a step along a direction that only
rounding sees would not)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eta", [0.3, 0.6])
@pytest.mark.parametrize("inner", [20, 64, 300])
def test_contradicting_rows(eta, inner):
    import paper_2509_19267_amd as rg
    m, n = 50, 20
    a = np.zeros((m, n))
    v = np.random.default_rng(1).standard_normal(m)
    for i in range(m):
        a[i, 4 * (i % 5):4 * (i % 5) + 4] = v[i]     # equal columns in fours
    rp = np.arange(0, 4 * m + 1, 4, dtype=np.int64)
    ci = (4 * (np.repeat(np.arange(m), 4) % 5) + np.tile(np.arange(4), m))
    csr = (torch.as_tensor(rp).cuda(),
           torch.as_tensor(ci.astype(np.int32)).cuda(),
           torch.as_tensor(a[np.repeat(np.arange(m), 4), ci]).cuda())
    for seed in range(60):
        s = rg.Solver(csr=csr, shape=(m, n), eta=eta, stop="none", max_iter=10,
                      inner_max=inner, inner_tol=1e-14, seed=seed,
                      sparse_cg=True)
        g = torch.Generator(device="cuda").manual_seed(seed + 100)
        b = torch.randn(n, generator=g, dtype=torch.float64, device="cuda")
        w, _ = s.solve_adjoint(b)                    # raises on a NaN weight
        s.close()
        assert torch.isfinite(w).all(), seed

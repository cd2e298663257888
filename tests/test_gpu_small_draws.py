"""Draws by one workgroup where the number of weights per thread changes (up to
1024, 2048, 4096, more), with ties across the candidates that four threads each
rank, and zeros: bit for bit the oracle's.  And a batch of one system, whose
list one workgroup writes in passes of 16384, against the same system alone,
drawn by many workgroups: a diagonal matrix, whose solution shows every index
drawn; both divide each entry alike, 1e-12 leaves room for the CG's rounding."""
import numpy as np
import pytest
import torch

from oracle.select import select as oselect

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 3, 5, 1023, 1024, 1025, 2047, 2048, 2049,
                               4095, 4096, 4097])
def test_bit_exact(d):
    import paper_2509_19267_amd as rg
    rng = np.random.default_rng(d)
    plain = rng.random(d)
    zeros = np.where(rng.random(d) < 0.4, 0.0, plain)
    # keys above the range: infinite keys, all equal
    ties = np.where(rng.random(d) < 0.5, 5e-324, 1e-300)
    for e in (plain, zeros, ties):
        for k in {1, max(1, d // 7), max(1, d // 2), d}:
            got = rg.select(torch.as_tensor(e).cuda(), k, seed=7, it=d,
                            phase=1).cpu().numpy()
            assert np.array_equal(got.astype(np.int64),
                                  oselect(e, k, 7, d, 1)), k


@pytest.mark.parametrize("n", [4097, 16384, 16385, 40000])
def test_one_system_batch(n):
    import paper_2509_19267_amd as rg
    rng = np.random.default_rng(n)
    csr = (torch.arange(n + 1, dtype=torch.int64).cuda(),
           torch.arange(n, dtype=torch.int32).cuda(),
           torch.as_tensor(rng.uniform(1.0, 2.0, n)).cuda())
    b = torch.as_tensor(rng.standard_normal(n)).cuda()
    kw = dict(k_col=n // 4, k_row=n // 3, stop="none", max_iter=2, seed=5)
    one = rg.Solver(csr=csr, shape=(n, n), sparse_cg=True, **kw)
    bat = rg.BatchSolver(csr, np.array([0, n]), np.array([0, n]), **kw)
    x, y = one.solve(b)[0], bat.solve(b)[0]
    one.close()
    bat.close()
    assert torch.equal(x != 0, y != 0) and int((x != 0).sum()) >= n // 3
    assert (x - y).norm() <= 1e-12 * x.norm()

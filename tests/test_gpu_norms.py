"""The norms of the stop tests (whole system and per system of a batch) where
their reductions change shape: one element, around one round of a workgroup's
loads, several rounds, one and many workgroups.  RSE of a resumed solve's first
test is ||b - A x||^2 / ||b||^2 for the given x whatever z is.  A thread adds
at most len / 1024 + 40 squares of one sign, r + z rounds twice more: within
1e-13 of the quotient (eps 1.1e-16)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 1023, 1025, 8191, 8193, 30000]


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _diag(n, rng):
    d = rng.uniform(1.0, 2.0, n)
    csr = (torch.arange(n + 1, dtype=torch.int64).cuda(),
           torch.arange(n, dtype=torch.int32).cuda(), torch.as_tensor(d).cuda())
    return d, csr, rng.standard_normal(n), rng.standard_normal(n)


def _resume(s, b, x):
    dev = [torch.as_tensor(v.copy()).cuda() for v in (b, x, 0.0 * b)]
    return s.solve_resume(dev[0], dev[1], dev[2], 0)


@pytest.mark.parametrize("n", SIZES + [2000000])
def test_whole(rg, n):
    d, csr, x, b = _diag(n, np.random.default_rng(n))
    s = rg.Solver(csr=csr, shape=(n, n), eta=0.1, stop="rse", tol=1e30,
                  max_iter=1, sparse_cg=True)
    info = _resume(s, b, x)
    s.close()
    want = np.sum((b - d * x) ** 2) / np.sum(b ** 2)
    got = (info[-1] if isinstance(info, tuple) else info)["final_metric"]
    print(n, got, want, flush=True)
    assert abs(got - want) <= 1e-13 * want


def test_batch(rg):
    off = np.concatenate([[0], np.cumsum(SIZES)])
    d, csr, x, b = _diag(int(off[-1]), np.random.default_rng(1))
    s = rg.BatchSolver(csr, off, off, eta=0.1, stop="rse", tol=1e30,
                       max_iter=1)
    _resume(s, b, x)
    met = s.batch_info()[1]
    s.close()
    for i in range(len(SIZES)):
        q = slice(off[i], off[i + 1])
        want = np.sum((b - d * x)[q] ** 2) / np.sum(b[q] ** 2)
        print(SIZES[i], met[i], want, flush=True)
        assert abs(met[i] - want) <= 1e-13 * want

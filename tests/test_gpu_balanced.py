"""Sparse CG products balanced by nonzeros, against the row-split ones
(cg_split) after the same number of CG steps: rows longer than a workgroup's
tile and than its span, runs of empty rows at the start, between and at the
end, a full column, fewer nonzeros than one workgroup takes and spans that end
inside a row.  The same operations with sums in another order: three CG steps
on rows of unit norm grow rounding by a few hundred at most, so 1e-11 of the
norm (eps 1.1e-16).  In the mixed form (FP32 products) the refined solution of
a consistent system, to the stated 1e-9."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _system(m, n, mean, longs, gap, seed):
    rng = np.random.default_rng(seed)
    ln = np.minimum(n, 1 + rng.geometric(1.0 / mean, m))
    ln[rng.choice(m, len(longs), False)] = np.minimum(n, longs)
    ln[:gap] = 0
    ln[m // 2:m // 2 + gap] = 0
    ln[m - gap:] = 0
    rows = [np.sort(rng.choice(n, k, False)) for k in ln]
    for r in range(gap, m // 2, 3):                      # a full column
        if ln[r] and rows[r][0] != 0:
            rows[r][0] = 0
    rp = np.concatenate([[0], np.cumsum(ln)])
    ci = np.concatenate(rows)
    v = rng.standard_normal(len(ci))
    r = np.repeat(np.arange(m), ln)
    v /= np.sqrt(np.bincount(r, v * v, m))[r]
    x = rng.standard_normal(n)
    ax = np.bincount(r, v * x[ci], m)
    csr = (torch.as_tensor(rp.astype(np.int64)).cuda(),
           torch.as_tensor(ci.astype(np.int32)).cuda(),
           torch.as_tensor(v).cuda())
    return csr, ax, x, rng


SHAPES = [(120, 100, 2, [90], 3, 40, 50), (700, 600, 4, [600, 550], 40, 200, 300),
          (5000, 3000, 10, [3000, 1500, 1024, 1025, 2048], 300, 900, 1500),
          (30000, 12000, 7, [9000, 5000, 300], 1000, 6000, 9000),
          (3000, 20000, 9, [20000], 1, 4000, 1500)]


@pytest.mark.parametrize("m,n,mean,longs,gap,kc,kr", SHAPES)
def test_steps(rg, m, n, mean, longs, gap, kc, kr):
    csr, ax, _, rng = _system(m, n, mean, longs, gap, m + n)
    b = torch.as_tensor(ax + 0.1 * rng.standard_normal(m)).cuda()
    out = []
    for split in (False, True, False):
        s = rg.Solver(csr=csr, shape=(m, n), k_col=kc, k_row=kr, stop="none",
                      max_iter=2, seed=3, inner_max=3, inner_tol=1e-14,
                      sparse_cg=True, cg_split=split, graph_iters=1)
        x, _ = s.solve(b)
        out.append((x.clone(), s.get_z().clone()))
        s.close()
    for got, want, again in zip(*out):
        d = (got - want).norm().item()
        print(m, n, d, want.norm().item(), flush=True)
        assert d <= 1e-11 * want.norm().item()
        assert torch.equal(got, again)


def test_mixed(rg):
    m, n = 6000, 2000
    csr, ax, x, _ = _system(m, n, 8, [2000, 1500, 700], 100, 5)
    x = torch.as_tensor(x).cuda()
    s = rg.Solver(csr=csr, shape=(m, n), k_col=900, k_row=1500,
                  precision="mixed_f32", stop="err_ref", tol=1e-9,
                  max_iter=20000, sparse_cg=True)
    got, info = s.solve(torch.as_tensor(ax).cuda(), x_ref=x)
    s.close()
    print(info, ((got - x).norm() / x.norm()).item(), flush=True)
    assert (got - x).norm() <= 1e-9 * x.norm()

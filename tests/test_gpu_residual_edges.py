"""The nonzero-balanced residual pass where the last row (and column) runs
through chunks of 256 nonzeros that own no rows, at row counts whose pointer
array fills whole pages.  Against FP64 products on the CPU within the usual
sum bound, (entries per row) * eps * |A| |x|, with a factor of 2."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,tail", [(1, 700), (2, 257), (511, 256), (511, 900),
                                    (1023, 2000)])
@pytest.mark.parametrize("transpose", [False, True])
def test_long_last_row(m, tail, transpose):
    import paper_2509_19267_amd as rg
    n = 2048
    rng = np.random.default_rng(m + tail)
    a = np.zeros((m, n))
    a[np.arange(m - 1), rng.integers(0, n, m - 1)] = rng.standard_normal(m - 1)
    a[m - 1, rng.choice(n, tail, False)] = rng.standard_normal(tail)
    a = a.T.copy() if transpose else a
    rp = np.concatenate([[0], np.cumsum((a != 0).sum(1))])
    r, c = np.nonzero(a)
    s = rg.Solver(csr=(torch.as_tensor(rp.astype(np.int64)).cuda(),
                       torch.as_tensor(c.astype(np.int32)).cuda(),
                       torch.as_tensor(a[r, c]).cuda()),
                  shape=a.shape, k_col=1, k_row=1, sparse_cg=True)
    x, z = rng.standard_normal(a.shape[1]), rng.standard_normal(a.shape[0])
    ax, atz = s.apply(torch.as_tensor(x).cuda(), torch.as_tensor(z).cuda())
    ax, atz = ax.cpu().numpy(), atz.cpu().numpy()
    s.close()
    for got, mm, v in ((ax, a, x), (atz, a.T, z)):
        bound = 2 * (1 + (mm != 0).sum(1)) * 2.3e-16 * (np.abs(mm) @ np.abs(v))
        assert (np.abs(got - mm @ v) <= bound).all()

"""Products of a matrix with many right-hand sides in row groups (rows that
share columns): against dense FP64 products, on banded matrices with a last
group of every size, empty rows and rows that share nothing, right-hand-side
counts around one and two waves.  Tolerances: the usual sum bound,
(entries per row) * eps * |A| |x|, with a factor of 2."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _banded(m, n, seed):
    rng = np.random.default_rng(seed)
    a = np.zeros((m, n))
    for i in range(m):
        if i % 17 == 5:
            continue                                   # an empty row
        c0 = min(max(0, i * n // m - 10 + rng.integers(0, 2)), n - 1)
        w = rng.integers(18, 24)
        a[i, c0:c0 + w] = rng.standard_normal(min(w, n - c0))
        if i % 13 == 0:
            a[i, :] = 0.0
            a[i, rng.integers(0, n)] = 1.5             # shares nothing
    return a


def _csr(a):
    rp = np.concatenate([[0], np.cumsum((a != 0).sum(1))]).astype(np.int64)
    r, c = np.nonzero(a)
    return (torch.as_tensor(rp).cuda(), torch.as_tensor(c.astype(np.int32)).cuda(),
            torch.as_tensor(a[r, c]).cuda())


@pytest.mark.parametrize("m,n", [(120, 100), (121, 100), (122, 61), (123, 64),
                                 (7, 5), (64, 300)])
@pytest.mark.parametrize("R", [33, 64, 70, 128])
def test_products(rg, m, n, R):
    a = _banded(m, n, m + R)
    a32 = a.astype(np.float32).astype(np.float64)
    s = rg.MultiRhsSolver(_csr(a), (m, n), R, precision="mixed_f32")
    rng = np.random.default_rng(R)
    x, z = rng.standard_normal((R, n)), rng.standard_normal((R, m))
    for prec, mat, eps in (("f64", a, 2.3e-16), ("f32", a32, 1.2e-7)):
        dt = torch.float64 if prec == "f64" else torch.float32
        xv = torch.as_tensor(x).to(dt).cuda()
        zv = torch.as_tensor(z).to(dt).cuda()
        ax, atz = s.apply(xv.reshape(-1), zv.reshape(-1), precision=prec)
        xd, zd = xv.double().cpu().numpy(), zv.double().cpu().numpy()
        for got, v, mm in ((ax, xd, mat), (atz, zd, mat.T)):
            bound = 2 * (1 + (mm != 0).sum(1)) * eps * (np.abs(v) @ np.abs(mm).T)
            err = np.abs(got.double().cpu().numpy().reshape(R, -1) - v @ mm.T)
            assert (err <= bound).all()
    s.close()


def test_infinity_stays_in_its_rows(rg):
    """A column that a row does not hold does not reach it, whatever its
    value: groups make no products with absent entries."""
    m, n, R = 96, 90, 64
    a = _banded(m, n, 1)
    s = rg.MultiRhsSolver(_csr(a), (m, n), R)
    x = np.ones((R, n))
    x[3, 40] = np.inf
    x[5, 41] = np.nan
    ax, _ = s.apply(torch.as_tensor(x).cuda().reshape(-1),
                    torch.zeros(R * m, dtype=torch.float64, device="cuda"))
    ax = ax.cpu().numpy().reshape(R, m)
    s.close()
    assert (np.isfinite(ax[3]) == (a[:, 40] == 0)).all()
    assert (np.isnan(ax[5]) == (a[:, 41] != 0)).all()
    keep = np.ones(R, bool)
    keep[[3, 5]] = False
    assert np.isfinite(ax[keep]).all()

"""Products in row groups at sizes that take them in both precisions (2800
gathers of 64 values a compute unit): banded matrices with a last group of
every size, empty rows, rows that share nothing and a full row,
right-hand-side counts around one to four waves.  Against sparse FP64 products
on the CPU within the usual sum bound, (entries per row) * eps * |A| |x|, with
a factor of 2.  And an entry that is finite in FP64 and infinite in FP32
reaches only the row that holds it: neither the other rows of its group nor
those whose columns are read past the end of a list."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu


def _banded(m, n, seed, full):
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    for i in range(m):
        if i % 17 == 5:
            continue                                   # an empty row
        c0 = min(max(0, i * n // m - 10 + int(rng.integers(0, 2))), n - 1)
        c = np.arange(c0, min(n, c0 + int(rng.integers(18, 24))))
        if i % 13 == 0:
            c = rng.integers(0, n, 1)                  # shares nothing
        if full and i == m // 2:
            c = np.arange(n)
        rows.append(np.full(len(c), i))
        cols.append(c)
    r, c = np.concatenate(rows), np.concatenate(cols)
    a = sp.csr_matrix((rng.standard_normal(len(r)), (r, c)), shape=(m, n))
    a.sort_indices()
    return a


def _dev(a):
    return (torch.as_tensor(a.indptr.astype(np.int64)).cuda(),
            torch.as_tensor(a.indices.astype(np.int32)).cuda(),
            torch.as_tensor(a.data).cuda())


def _check(got, mat, v, eps, keep=slice(None)):
    cnt = np.diff(mat.indptr)
    bound = 2 * (1 + cnt) * eps * (abs(mat) @ np.abs(v).T).T
    err = np.abs(got.double().cpu().numpy().reshape(v.shape[0], -1) - (mat @ v.T).T)
    assert (err <= bound)[:, keep].all()


@pytest.mark.parametrize("m,n,R", [(42000, 42000, 33), (42001, 43000, 64),
                                   (42002, 42100, 64), (21003, 21003, 70),
                                   (21005, 21003, 128), (10502, 10501, 256)])
@pytest.mark.parametrize("full", [False, True])
def test_products(m, n, R, full):
    import paper_2509_19267_amd as rg
    a = _banded(m, n, m + R, full)
    s = rg.MultiRhsSolver(_dev(a), (m, n), R, precision="mixed_f32")
    rng = np.random.default_rng(R)
    x, z = rng.standard_normal((R, n)), rng.standard_normal((R, m))
    for prec, np_t, eps in (("f64", np.float64, 2.3e-16),
                            ("f32", np.float32, 1.2e-7)):
        xv, zv = x.astype(np_t), z.astype(np_t)
        mat = a.astype(np_t).astype(np.float64)
        ax, atz = s.apply(torch.as_tensor(xv).reshape(-1).cuda(),
                          torch.as_tensor(zv).reshape(-1).cuda(), precision=prec)
        _check(ax, mat, xv.astype(np.float64), eps)
        _check(atz, mat.T.tocsr(), zv.astype(np.float64), eps)
    s.close()


@pytest.mark.parametrize("R", [33, 64, 70])
@pytest.mark.parametrize("row", [4, 5, 6, 7, 4000, 32998])
def test_infinite_in_fp32(R, row):
    import paper_2509_19267_amd as rg
    m, n = (66000, 66000) if R <= 64 else (33000, 33000)
    i = np.repeat(np.arange(m), 12)
    j = np.tile(np.arange(12), m) + i
    rng = np.random.default_rng(row)
    ok = (j < n) & ((j - i < 10) | (j - i - 9 <= i % 3))
    a = sp.csr_matrix((rng.standard_normal(ok.sum()), (i[ok], j[ok])), shape=(m, n))
    col = min(row + 3, n - 1)
    a[row, col] = 1e300
    a.sort_indices()
    s = rg.MultiRhsSolver(_dev(a), (m, n), R, precision="mixed_f32")
    x = rng.standard_normal((R, n)).astype(np.float32)
    z = rng.standard_normal((R, m)).astype(np.float32)
    ax, atz = s.apply(torch.as_tensor(x).reshape(-1).cuda(),
                      torch.as_tensor(z).reshape(-1).cuda(), precision="f32")
    s.close()
    a[row, col] = 0.0
    b = a.astype(np.float32).astype(np.float64)
    for got, v, mat, hit in ((ax, x, b, row), (atz, z, b.T.tocsr(), col)):
        assert not torch.isfinite(got.reshape(R, -1)[:, hit]).any()
        keep = np.arange(mat.shape[0]) != hit
        _check(got, mat, v.astype(np.float64), 1.2e-7, keep)

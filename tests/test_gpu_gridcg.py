"""Sparse block projections in one launch, against the same projections with
a launch per CG phase (cg_split) after the same number of steps: one and many
workgroups, several segments per lane group, lane groups of 1 to 64, rows
longer than what a lane keeps, empty rows and columns, row blocks wider and
taller than A.  Both sides do the same operations with sums in another order;
three CG steps on blocks of unit rows grow rounding by a few hundred at most,
so 1e-11 of the norm (eps 1.1e-16).  And two solves at the same time on two
streams, whose workgroups may not all fit the device together: the bits of
the solves alone."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import paper_2509_19267_amd as m
    return m


def _system(m, n, per_row, seed):
    rng = np.random.default_rng(seed)
    rows = [np.sort(rng.choice(n, min(n, max(0, int(per_row * f))), False))
            if i % 23 != 11 else np.zeros(0, int)        # some rows are empty
            for i, f in enumerate(rng.uniform(0.3, 1.7, m))]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    ci = np.concatenate(rows).astype(np.int32)
    v = rng.standard_normal(len(ci))
    lens = np.repeat(np.diff(rp), np.diff(rp))
    v /= np.sqrt(np.maximum(lens, 1))
    ax = np.add.reduceat(np.concatenate([v * rng.standard_normal(n)[ci], [0.]]),
                         np.minimum(rp[:-1], len(ci))) * (np.diff(rp) > 0)
    csr = (torch.as_tensor(rp.astype(np.int64)).cuda(),
           torch.as_tensor(ci).cuda(), torch.as_tensor(v).cuda())
    return csr, torch.as_tensor(ax + 0.1 * rng.standard_normal(m)).cuda()


SHAPES = [(3, 2, 2, 1, 1), (40, 30, 3, 11, 17), (513, 130, 9, 65, 100),
          (700, 900, 40, 300, 350), (2000, 1500, 150, 700, 600),
          (45000, 30000, 5, 20000, 24000), (2600, 60, 20, 30, 1300),
          (9000, 700, 40, 350, 4500), (60000, 300, 2, 150, 30000)]


@pytest.mark.parametrize("m,n,per_row,kc,kr", SHAPES)
def test_steps(rg, m, n, per_row, kc, kr):
    csr, b = _system(m, n, per_row, m + n)
    out = []
    for split in (False, True):
        s = rg.Solver(csr=csr, shape=(m, n), k_col=kc, k_row=kr, stop="none",
                      max_iter=2, seed=3, inner_max=3, inner_tol=1e-14,
                      sparse_cg=True, cg_split=split, graph_iters=1)
        x, info = s.solve(b)
        out.append((x.clone(), s.get_z().clone()))
        s.close()
    for got, want in zip(*out):
        d = (got - want).norm().item()
        print(m, n, d, want.norm().item(), flush=True)
        assert d <= 1e-11 * want.norm().item()


@pytest.mark.parametrize("m,n,per_row,kc,kr", SHAPES[3:8])
def test_two_streams(rg, m, n, per_row, kc, kr):
    handles = []
    for i in range(2):
        csr, b = _system(m, n, per_row, m + i)
        st = torch.cuda.Stream()
        handles.append((rg.Solver(csr=csr, shape=(m, n), k_col=kc, k_row=kr,
                                  stop="none", max_iter=6, seed=i,
                                  inner_max=5, sparse_cg=True, stream=st), b,
                        st))
    torch.cuda.synchronize()

    def solve(i, out):
        s, b, st = handles[i]
        with torch.cuda.stream(st):
            x, _ = s.solve(b)
            out[i] = x.clone()
            st.synchronize()

    alone, both = {}, {}
    for i in range(2):
        solve(i, alone)
    ts = [threading.Thread(target=solve, args=(i, both)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in range(2):
        assert torch.equal(alone[i], both[i])
        handles[i][0].close()

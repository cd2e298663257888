"""One large system beside many tiny ones, where the lists of the blocks are
written by fewer workgroups than the largest system would have.  After one
iteration the equations of every system's own draws hold (A_U^T z = 0 and
A^J x = (b - z)^J for the sets that the draw alone gives with the system's id):
systems I + E with |E| < 0.6, so condition numbers below 16 for the Grams, CG
to 1e-14 of the whole norm (250), 1e-9 for a system of norm 1."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu


def _system(n, per, rng):
    r = np.repeat(np.arange(n), per)
    e = sp.csr_matrix((rng.uniform(-1, 1, n * per), (r, rng.integers(0, n, n * per))),
                      shape=(n, n))
    e *= 0.3 / max(abs(e).sum(0).max(), abs(e).sum(1).max())
    return sp.identity(n, format="csr") + e


@pytest.mark.parametrize("tiny", [60, 900, 2500])
def test_draws_reach_their_systems(tiny):
    import paper_2509_19267_amd as rg
    rng = np.random.default_rng(tiny)
    sizes = [40] * 2 + [60000] + [6] * tiny
    mats = [_system(n, min(3, n), rng) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    a = sp.block_diag(mats, format="csr")
    a.sort_indices()
    b = rng.standard_normal(off[-1])
    s = rg.BatchSolver((torch.as_tensor(a.indptr.astype(np.int64)).cuda(),
                        torch.as_tensor(a.indices.astype(np.int32)).cuda(),
                        torch.as_tensor(a.data).cuda()), off, off, eta=0.5,
                       stop="none", max_iter=1, inner_max=80, inner_tol=1e-14,
                       graph_iters=1, seed=9)
    x, _ = s.solve(torch.as_tensor(b).cuda())
    x, z = x.cpu().numpy(), s.get_z().cpu().numpy()
    s.close()
    for i in [0, 1, 2, 3, 4, 30, tiny // 2, tiny, tiny + 2]:
        q, m, k = slice(off[i], off[i + 1]), mats[i], sizes[i] // 2
        def draw(w, phase):
            return rg.select(torch.as_tensor(w).cuda(), k, seed=9, phase=phase,
                             sys=i).cpu().numpy()
        g = m.T @ b[q]
        u = draw(g ** 2 / np.asarray(m.multiply(m).sum(0)).ravel(), 0)
        r = b[q] - z[q]
        j = draw(r ** 2 / np.asarray(m.multiply(m).sum(1)).ravel(), 1)
        assert len(u) == len(j) == k
        assert np.linalg.norm((m.T @ z[q])[u]) <= 1e-9 * max(1.0, np.linalg.norm(g))
        assert np.linalg.norm((m @ x[q] - r)[j]) <= 1e-9 * max(1.0, np.linalg.norm(r))

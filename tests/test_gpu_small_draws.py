"""Draws by one workgroup where the number of weights per thread changes (up to
1024, 2048, 4096, more), with ties across the candidates that four threads each
rank, and zeros: bit for bit the oracle's."""
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

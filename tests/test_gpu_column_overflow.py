"""A sparse column block whose CG overflows: the sum of q^2 is infinite in the
first step and NaN in the second.  No step is taken then, so z changes in no
row that the block does not touch (a step of NaN would write NaN to all), and
the solve reports the numeric error that the next weights show.  In each form
of the block CG: one launch, balanced by nonzeros, a launch per phase."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("long_row", [False, True])
@pytest.mark.parametrize("split", [False, True])
def test_rows_off_the_block(long_row, split):
    import paper_2509_19267_amd as rg
    n = 200
    # rows 0-99: one entry each in column i; rows 100-199 likewise, but b = 0
    # there, so their columns have no weight; column 0 is huge
    rows = [[i] for i in range(n)]
    if long_row:
        rows[1] = list(range(1, 100))
    rp = [0]
    for r in rows:
        rp.append(rp[-1] + len(r))
    v = torch.ones(rp[-1], dtype=torch.float64)
    v[0] = 1e150
    b = torch.zeros(n, dtype=torch.float64)
    b[:100] = 1.0
    b[0] = 1e3
    s = rg.Solver(csr=(torch.tensor(rp).cuda(),
                       torch.tensor(sum(rows, []), dtype=torch.int32).cuda(),
                       v.cuda()), shape=(n, n), k_col=100, k_row=50,
                  stop="none", max_iter=1, inner_max=4, sparse_cg=True,
                  cg_split=split, graph_iters=1)
    with pytest.raises(rg.RgdbekError) as e:
        s.solve(b.cuda())
    assert e.value.status == rg._binding.ERR_NUMERIC
    z = s.get_z().cpu()
    s.close()
    assert not torch.isfinite(z[:100]).all()
    assert (z[100:] == 0).all()

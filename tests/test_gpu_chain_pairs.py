"""Chain pairs (a TRSM and the next POTRF in one workgroup) on the GPU: widths
with one tile below the diagonal and with several, a last tile row of every
kind of remainder, both tile sizes and both launches; with one, two and three
workgroups, where a workgroup takes every ticket behind a pair's own wait.
Factor, solution and log-determinant against the oracle: 1e-12; and bitwise
the same for every number of workgroups."""
import pytest

import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import oracle_reference, rel, say, to_device_cols

pytestmark = pytest.mark.gpu

TF_CHAIN = 1 << 13


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("n,arrow,width", [(130, 0, 40), (641, 3, 20), (900, 40, 64), (1200, 0, [30, 180]), (1503, 70, 140)])
def test_pairs_match_oracle(tile, n, arrow, width):
    import torch
    p = I.make_pattern(n, arrow, width, seg=300)
    vals = I.make_values(p, seed=n)
    B = I.rhs(p.N, 2, seed=5)
    ref = oracle_reference(p, vals, B)
    sym = S.Symbolic.from_pattern(p, tile=tile, ordering=S.STILES_ORDER_NONE)
    tasks = S.stiles_symbolic_export(sym.handle, "ftask").reshape(-1, 8)
    assert ((tasks[:, 0] & TF_CHAIN) != 0).any()
    dv = torch.from_numpy(vals).cuda()
    first = None
    for cap in (0, 1, 2, 3):
        say("[gpu chain pairs] T=%d n=%d a=%d w=%s workgroups %d" % (tile, n, arrow, width, cap))
        fac = S.Factor(sym, nrhs_max=2)
        if cap:
            fac.set_max_workgroups(cap)
        fac.factorize(dv)
        assert fac.info() == 0
        L = fac.extract()
        ld = fac.logdet().clone()
        X = to_device_cols(B)
        fac.factorize_solve(dv, X)
        assert torch.equal(fac.extract(), L)
        if first is None:
            first = (L.clone(), ld, X.clone())
            assert rel(L.cpu().numpy(), ref["L"]) <= 1e-12
            assert rel(X.cpu().numpy(), ref["X"]) <= 1e-12
            assert abs(ld.item() - ref["logdet"]) <= 1e-12 * abs(ref["logdet"])
        assert torch.equal(L, first[0]) and torch.equal(ld, first[1]) and torch.equal(X, first[2])

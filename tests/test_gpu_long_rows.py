"""Solves over long rows at the edges of their sums: arrow rows that meet
every tile column, whose partial products go through one slot per chunk
(counts of every remainder by eight), with chunks of one and more products,
one to sixteen right-hand sides, both tile sizes; separate and merged launch.
Solution against the oracle: 1e-12 (FP64 throughout), and the merged launch
bitwise the separate one."""
import pytest

import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import oracle_reference, rel, say, to_device_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("n,nrhs", [(2300, 1), (3400, 16), (4500, 5), (5600, 16), (6600, 3), (7400, 2), (9000, 7),
                                    (10200, 1), (12300, 4), (16600, 16)])
def test_long_rows(tile, n, nrhs):
    import torch
    p = I.make_pattern(n, 5, [20, 45], seg=700)
    vals = I.make_values(p, seed=n + tile)
    B = I.rhs(p.N, nrhs, seed=3)
    ref = oracle_reference(p, vals, B)
    sym = S.Symbolic.from_pattern(p, tile=tile, ordering=S.STILES_ORDER_NONE)
    tasks = S.stiles_symbolic_export(sym.handle, "stask").reshape(-1, 8)
    sums = tasks[(tasks[:, 0] & 0xff) == 13]
    assert len(sums) > 0
    say("[gpu long rows] T=%d n=%d nrhs=%d slots %s" % (tile, n, nrhs, sorted(set((sums[:, 3] - sums[:, 2]).tolist()))))
    dv = torch.from_numpy(vals).cuda()
    fac = S.Factor(sym, nrhs_max=nrhs)
    fac.factorize(dv)
    X = to_device_cols(B)
    fac.solve(X)
    assert rel(X.cpu().numpy(), ref["X"]) <= 1e-12
    Y = to_device_cols(B)
    fac.factorize_solve(dv, Y)
    assert torch.equal(X, Y)

"""The update products' operand ring at its edges: update tasks of one to
thirty-two products (the `chunk` option), so that the ring holds fewer stages
than slots, exactly as many, and many times over; both tile sizes; FP64 and
FP32 operands; partial sums of the arrow corner (with and without the tree).
Factor against the oracle: 1e-12 in FP64, 1e-5 with FP32 updates (their
rounding over sums of at most a few hundred products)."""
import numpy as np
import pytest

import oracle
import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import col_tile_err, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("precision,tol", [(S.STILES_FP64, 1e-12), (S.STILES_MIXED32, 1e-5)])
@pytest.mark.parametrize("chunk,ratio", [(1, 2), (2, 0), (3, 2), (4, 0), (5, 2), (12, 0), (32, 2)])
def test_update_chunks(tile, precision, tol, chunk, ratio):
    import torch
    p = I.make_pattern(1150, 70, [300, 90, 430], seg=400)
    vals = I.make_values(p, seed=chunk + tile)
    L_o, info = oracle.factor(p.f, vals, nthreads=8)
    assert info == 0
    say("[gpu update ring] T=%d chunk %d tree ratio %d precision %d" % (tile, chunk, ratio, precision))
    sym = S.Symbolic.from_pattern(p, tile=tile, chunk=chunk, tree_min_ratio=ratio)
    fac = S.Factor(sym, precision)
    dv = torch.from_numpy(vals).cuda()
    fac.factorize(dv)
    assert fac.info() == 0
    L = fac.extract()
    assert rel(L.cpu().numpy(), L_o) <= tol
    assert col_tile_err(L.cpu().numpy(), L_o, p.f, tile) <= tol
    fac.factorize(dv)                        # the same bits again
    assert torch.equal(fac.extract(), L)

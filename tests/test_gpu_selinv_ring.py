"""Selected-inversion products at the edges of their operand ring: tasks of
one to thirty-two products (the `chunk` option), so that the ring holds fewer
stages than slots, exactly as many, and many times over, with Sigma tiles read
as stored and transposed; both tile sizes, a last tile row of every kind of
remainder.  Selected entries against the oracle's recursion: 1e-12 normwise,
the bar of the other selected-inversion tests (FP64 throughout)."""
import numpy as np
import pytest

import oracle
import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("chunk", [1, 2, 3, 4, 5, 12, 32])
def test_selinv_chunks(tile, chunk):
    import torch
    p = I.make_pattern(1150 + 13 * chunk, 70, [300, 90, 430], seg=400)
    vals = I.make_values(p, seed=chunk + tile)
    L, info = oracle.factor(p.f, vals, nthreads=8)
    assert info == 0
    want = oracle.selinv(p.f, L, nthreads=8)
    say("[gpu selinv ring] T=%d chunk %d" % (tile, chunk))
    sym = S.Symbolic.from_pattern(p, tile=tile, chunk=chunk, ordering=S.STILES_ORDER_NONE)
    fac = S.Factor(sym)
    fac.factorize(torch.from_numpy(vals).cuda())
    si = S.SelInv(fac)
    si.compute()
    got = si.extract().cpu().numpy()
    assert rel(got, want) <= 1e-12
    d = si.diag().clone()
    rp = np.concatenate([[0], np.cumsum(np.arange(len(p.f)) - np.asarray(p.f) + 1)])
    assert np.max(np.abs(d.cpu().numpy() - want[rp[1:] - 1]) / want[rp[1:] - 1]) <= 1e-12
    si.compute()                             # the same bits again
    assert torch.equal(si.diag(), d)

"""The diagonal-tile factorization (16-column panels with the inverse built
beside them) at sizes around the panel and tile edges: a dense matrix of one
to three tile rows, its factor, solution (which uses the stored inverse) and
log-determinant against the oracle, and the reported column for a pivot that
fails at each place of a panel."""
import numpy as np
import pytest

import oracle
import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import oracle_reference, rel, say, to_device_cols

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 96, 129])
def test_dense_matrix_around_panel_and_tile_edges(n, tile):
    import torch
    p = I.make_pattern(n, 0, n)
    vals = I.make_values(p, seed=n)
    B = I.rhs(n, 2, seed=3)
    ref = oracle_reference(p, vals, B)
    say("[gpu diagonal tile] n=%d T=%d" % (n, tile))
    fac = S.Factor(S.Symbolic.from_pattern(p, tile=tile), nrhs_max=2)
    fac.factorize(torch.from_numpy(vals).cuda())
    assert fac.info() == 0
    X = to_device_cols(B)
    fac.solve(X)
    L_o, _ = oracle.factor(p.f, vals)
    assert rel(fac.extract().cpu().numpy(), L_o) <= TOL
    assert rel(X.cpu().numpy(), ref["X"]) <= TOL
    ld_o = oracle.logdet(p.f, L_o)
    assert abs(fac.logdet().item() - ld_o) <= TOL * max(1.0, abs(ld_o))


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("bad", [0, 1, 14, 15, 16, 31, 32, 47, 48, 63, 64, 70])
def test_failing_pivot_of_a_panel(bad, tile):
    import torch
    n = 71
    p = I.make_pattern(n, 0, n)
    vals = I.make_values(p, seed=5)
    vals[p.row_ptr()[bad + 1] - 1] = -1.0 if bad % 2 else 0.0
    _, info_o = oracle.factor(p.f, vals)
    say("[gpu diagonal tile] failing pivot %d T=%d" % (bad, tile))
    fac = S.Factor(S.Symbolic.from_pattern(p, tile=tile))
    fac.factorize(torch.from_numpy(vals).cuda())
    assert fac.info() == info_o == bad + 1


@pytest.mark.parametrize("tile", [32, 64])
def test_integer_factor_is_exact(tile):
    """A planted sparse factor of small integers with unit diagonal, whose
    tiles' inverses stay small: every product and sum is a whole number below
    2^53, so the factor comes back bit for bit."""
    import torch
    n = 150
    p = I.make_pattern(n, 0, n)
    rng = np.random.default_rng(11)
    L = np.tril(rng.choice([-1.0, 0.0, 1.0], p=[0.04, 0.92, 0.04], size=(n, n)), -1) + np.eye(n)
    A = L @ L.T
    big = max(np.abs(np.linalg.inv(L[i:i + tile, i:i + tile])).max() for i in range(0, n, tile))
    assert big ** 2 * np.abs(A).max() * n < 2.0 ** 53
    vals = np.concatenate([A[i, :i + 1] for i in range(n)])
    say("[gpu diagonal tile] integer factor T=%d" % tile)
    fac = S.Factor(S.Symbolic.from_pattern(p, tile=tile))
    fac.factorize(torch.from_numpy(vals).cuda())
    assert fac.info() == 0
    assert np.array_equal(fac.extract().cpu().numpy(), np.concatenate([L[i, :i + 1] for i in range(n)]))

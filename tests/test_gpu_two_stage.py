"""POTRF and TRSM tasks in their two-stage form under tickets of their own (no
chain pairs), on the GPU: plans with more work per workgroup than the pairing
rule allows, as the large matrices have them, at the smallest sizes that
reach it; both tile sizes, last tile rows with remainders, one to three
workgroups, the separate and the merged launch, FP64 and mixed precision.
Against the oracle: 1e-12; against a batch of the one matrix, whose waits are
single-stage: bitwise the same; the reported column for a pivot that fails at
each place of a panel; and launches abandoned inside the waits."""
import pytest

import oracle
import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

from gpu_util import oracle_reference, rel, rel_cols, say, to_device_cols
from permute_util import permute_profile

pytestmark = pytest.mark.gpu

TOL = 1e-12
TF_SPLIT, TF_CHAIN, POTRF = 1 << 11, 1 << 13, 4
CASES = {   # n, arrow, widths, segment, partitions
    32: (4003, 1001, [20, 84, 40], 450, 24),
    64: (12_011, 901, [32, 148, 70], 700, 24),
}


def make(tile):
    n, a, w, seg, parts = CASES[tile]
    p = I.make_pattern(n, a, w, seg=seg)
    sym = S.Symbolic.from_pattern(p, tile=tile, ordering=S.STILES_ORDER_ADAPTABLE_ND, nd_parts=parts)
    for name in ("ftask", "mtask"):
        tasks = S.stiles_symbolic_export(sym.handle, name).reshape(-1, 8)
        assert not (tasks[:, 0] & TF_CHAIN).any()
        two_stage = ((tasks[:, 0] & 0xff) == POTRF) & ((tasks[:, 0] & TF_SPLIT) != 0)
        assert two_stage.sum() >= 50
    return p, sym


@pytest.mark.parametrize("tile", [32, 64])
def test_two_stage_tasks_match_oracle(tile):
    import torch
    p, sym = make(tile)
    vals = I.make_values(p, seed=tile)
    B = I.rhs(p.N, 3, seed=5)
    ref = oracle_reference(p, vals, B)
    f2, v2 = permute_profile(p.f, vals, sym.perm())
    L2, info2 = oracle.factor(f2, v2, nthreads=8)
    assert info2 == 0
    dv = torch.from_numpy(vals).cuda()
    one = S.Factor(sym)
    S.Batch([one]).factorize([dv])
    L1 = one.extract()
    assert rel(L1.cpu().numpy(), L2) <= TOL
    first = None
    for cap in (0, 1, 2, 3):
        say("[gpu two stage] T=%d workgroups %d" % (tile, cap))
        fac = S.Factor(sym, nrhs_max=3)
        if cap:
            fac.set_max_workgroups(cap)
        fac.factorize(dv)
        assert fac.info() == 0
        assert torch.equal(fac.extract(), L1)
        ld = fac.logdet().clone()
        X = to_device_cols(B)
        fac.factorize_solve(dv, X)
        assert torch.equal(fac.extract(), L1)
        if first is None:
            first = (ld, X.clone())
            assert rel_cols(X.cpu().numpy(), ref["X"]) <= TOL
            assert abs(ld.item() - ref["logdet"]) <= TOL * abs(ref["logdet"])
        assert torch.equal(ld, first[0]) and torch.equal(X, first[1])


def make_paired(tile):
    p = I.make_pattern(3001, 33, [30, 150, 80], seg=700)
    sym = S.Symbolic.from_pattern(p, tile=tile, ordering=S.STILES_ORDER_NONE)
    assert (S.stiles_symbolic_export(sym.handle, "ftask").reshape(-1, 8)[:, 0] & TF_CHAIN).any()
    return p, sym


@pytest.mark.parametrize("tile,pairs", [(32, False), (64, False), (32, True), (64, True)])
def test_two_stage_mixed_precision(tile, pairs):
    import torch
    p, sym = make_paired(tile) if pairs else make(tile)
    vals = I.make_values(p, seed=tile + 1)
    B = I.rhs(p.N, 2, seed=6)
    ref = oracle_reference(p, vals, B)
    dv = torch.from_numpy(vals).cuda()
    one = S.Factor(sym, S.STILES_MIXED32)
    S.Batch([one]).factorize([dv])
    say("[gpu two stage] mixed T=%d" % tile)
    fac = S.Factor(sym, S.STILES_MIXED32, nrhs_max=2)
    X = to_device_cols(B)
    fac.factorize_solve(dv, X)
    assert fac.info() == 0
    assert torch.equal(fac.extract(), one.extract())
    assert rel_cols(X.cpu().numpy(), ref["X"]) <= TOL


@pytest.mark.parametrize("tile", [32, 64])
def test_two_stage_failing_pivots(tile):
    import torch
    p, sym = make(tile)
    good = I.make_values(p, seed=tile + 2)
    rp, perm = p.row_ptr(), sym.perm()
    fac = S.Factor(sym)
    base = 16 * tile                  # a tile row of the first partition
    rows = [base + q for q in (0, 1, 15, 16, 31, 32, 47, 48, 63) if q < tile]
    rows += [sym.info.N - 1, sym.info.n, sym.info.n - 1]
    for k, r in enumerate(rows):
        say("[gpu two stage] failing pivot %d T=%d" % (r, tile))
        vals = good.copy()
        vals[rp[perm[r] + 1] - 1] = -1.0 if k % 2 else 0.0
        fac.factorize(torch.from_numpy(vals).cuda())
        assert fac.info() == r + 1
        with pytest.raises(S.StilesError):   # no factor
            fac.logdet()
    fac.factorize(torch.from_numpy(good).cuda())
    assert fac.info() == 0


@pytest.mark.parametrize("tile,pairs", [(32, False), (64, False), (32, True), (64, True)])
def test_abandoned_launch_recovers(tile, pairs):
    """A deadline of one clock tick: the launch is abandoned inside the
    two-stage waits (of single tasks, or of chain pairs), and every counter is
    armed again for the next one."""
    import torch
    p, sym = make_paired(tile) if pairs else make(tile)
    dv = torch.from_numpy(I.make_values(p, seed=tile + 3)).cuda()
    B = to_device_cols(I.rhs(p.N, 1, seed=7))
    fac = S.Factor(sym)
    fac.factorize(dv)
    L = fac.extract().clone()
    X0 = B.clone()
    fac.factorize_solve(dv, X0)
    for merged in (False, True):
        say("[gpu two stage] one tick, T=%d pairs %d merged %d" % (tile, pairs, merged))
        X = B.clone()
        fac.set_wait_limit(1e-8)
        if merged:
            fac.factorize_solve(dv, X)
        else:
            fac.factorize(dv)
        torch.cuda.synchronize()
        with pytest.raises(S.StilesError) as e:
            fac.info()
        assert e.value.status == S.STILES_ETIMEOUT
        fac.set_wait_limit(0)
        for _ in range(2):
            X = B.clone()
            fac.factorize_solve(dv, X)
            assert fac.info() == 0
            assert torch.equal(fac.extract(), L) and torch.equal(X, X0)
            fac.factorize(dv)
            assert torch.equal(fac.extract(), L)

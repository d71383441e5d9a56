"""Chain pairs of the factorization (TF_CHAIN): a TRSM and the POTRF that its
workgroup runs next.  In every plan (natural order, adaptable ND, update
blocks; tickets by earliest start and by list schedules; factorization and
merged DAG) the POTRF is the TRSM's first successor and waits late for it, its
one fused operand is the TRSM's tile, and all its other predecessors have
earlier tickets than the TRSM, so that a workgroup never waits for a later
ticket.  Narrow bands in natural order pair every step of the chain."""
import numpy as np
import pytest

import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I
import dag_emulator as E

TF_CHAIN = 1 << 13


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("kw", [dict(ordering=S.STILES_ORDER_NONE), dict(ordering=S.STILES_ORDER_NONE, ublock=3),
                                dict(ordering=S.STILES_ORDER_ADAPTABLE_ND, nd_parts=3)], ids=["natural", "blocks", "nd"])
@pytest.mark.parametrize("sched_workers", [-1, 0, 16])
def test_pairs(tile, kw, sched_workers):
    p = I.make_pattern(2300, 24, [20, 150, 260], seg=500)
    sym = S.Symbolic.from_pattern(p, tile=tile, sched_workers=sched_workers, **kw)
    ex = lambda k: S.stiles_symbolic_export(sym.handle, k)
    for names in (("ftask", "fsucc", "fpairs"), ("mtask", "msucc", "mpairs")):
        tasks, succ, pairs = ex(names[0]).reshape(-1, 8), ex(names[1]), ex(names[2]).reshape(-1, 2)
        typ = tasks[:, 0] & 0xff
        preds = [[] for _ in range(len(tasks))]
        for t in range(len(tasks)):
            for q in range(tasks[t, 5], tasks[t, 6]):
                preds[E.succ_edge(succ[q])[0]].append((t, E.succ_edge(succ[q])[1]))
        paired = 0
        for t in np.nonzero((tasks[:, 0] & TF_CHAIN) != 0)[0]:
            assert typ[t] in (E.POTRF, E.TRSM)
            if typ[t] == E.POTRF:
                continue
            y, dec = E.succ_edge(succ[tasks[t, 5]])
            assert typ[y] == E.POTRF and tasks[y, 0] & TF_CHAIN and dec == 1
            assert tasks[t, 0] & E.TF_SPLIT and tasks[y, 0] & E.TF_SPLIT
            assert tasks[y, 4] - tasks[y, 3] == 1 and (pairs[tasks[y, 3]] == tasks[t, 1]).all()
            assert all(x < t for x, _ in preds[y] if x != t)
            paired += 1
        assert paired == int((((tasks[:, 0] & TF_CHAIN) != 0) & (typ == E.POTRF)).sum())
        if "nd_parts" not in kw:
            assert paired > 0


def test_narrow_band_pairs_every_step():
    p = I.make_pattern(2000, 8, 40)
    for tile in (32, 64):
        sym = S.Symbolic.from_pattern(p, tile=tile, ordering=S.STILES_ORDER_NONE)
        tasks = S.stiles_symbolic_export(sym.handle, "ftask").reshape(-1, 8)
        potrf = tasks[(tasks[:, 0] & 0xff) == E.POTRF]
        fused = potrf[:, 4] > potrf[:, 3]
        assert ((potrf[fused, 0] & TF_CHAIN) != 0).all() and fused.sum() >= len(potrf) - 2


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("sched_workers", [-1, 0, 16])
def test_nd_plans_have_pairs(tile, sched_workers):
    """The checks of test_pairs are not empty under adaptable ND."""
    p = I.make_pattern(2300, 24, [20, 150, 260], seg=500)
    sym = S.Symbolic.from_pattern(p, tile=tile, sched_workers=sched_workers, ordering=S.STILES_ORDER_ADAPTABLE_ND,
                                  nd_parts=3)
    assert sym.info.nd_parts == 3
    for name in ("ftask", "mtask"):
        tasks = S.stiles_symbolic_export(sym.handle, name).reshape(-1, 8)
        assert ((tasks[:, 0] & (0xff | TF_CHAIN)) == (E.TRSM | TF_CHAIN)).sum() >= 5

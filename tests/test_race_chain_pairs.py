"""Chain pairs of the factorization under ThreadSanitizer (host, no GPU): the
TRSM that stages the next POTRF's tile, hands its result on in the worker's own
memory and notifies its other successors from inside that POTRF, in the
factorization and the merged DAG; and the same plans with every task under its
own ticket, as a plan without pairs runs them.  Planted mistakes (a missing
edge into a pair or out of one, a notification before the result is stored, a
tile staged without a wait) are reported."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2501_02483_amd as S
from paper_2501_02483_amd import inputs as I

import dag_emulator as E
from test_race_emulator import TSAN_OPTIONS, _export, _export_merged, _oracle_factor_permuted, _run, exe  # noqa: F401

CASES = [
    # n, arrow, widths, segment, tile, ordering, parts
    (900, 40, [15, 70, 130], 300, 32, S.STILES_ORDER_NONE, 0),
    (1500, 24, [20, 60, 135], 500, 32, S.STILES_ORDER_ADAPTABLE_ND, 3),
    (700, 0, [20, 150], 350, 64, S.STILES_ORDER_NONE, 0),
]


def _plan(case):
    n, a, w, seg, T, ordering, parts = case
    p = I.make_pattern(n, a, w, seg=seg)
    vals = I.make_values(p, seed=n + a)
    plan = E.Plan(S.Symbolic.from_pattern(p, tile=T, ordering=ordering, nd_parts=parts))
    return p, vals, plan, I.to_dense(p, vals)[np.ix_(plan.perm, plan.perm)]


def _strip(path, ntasks):
    """Takes the pair flags out of an exported plan."""
    with open(path, "r+b") as f:
        f.seek(7 * 4)
        w = np.frombuffer(f.read(ntasks * 32), dtype=np.int32).reshape(-1, 8).copy()
        w[:, 0] &= ~E.TF_CHAIN
        f.seek(7 * 4)
        f.write(w.tobytes())


def _check(exe, tmp_path, ntasks, compare):
    inp, out = str(tmp_path / "plan.bin"), str(tmp_path / "out.bin")
    for pairs in (True, False):
        if not pairs:
            _strip(inp, ntasks)
        for seed in (1, 2, 3):
            r = _run(exe, inp, out, seed)
            assert r.returncode == 0, (pairs, r.stderr[-3000:])
            assert "ThreadSanitizer" not in r.stderr
            compare(np.fromfile(out, dtype=np.float64))


def _err(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("case", CASES, ids=["natural", "nd3", "T64"])
def test_pairs_have_no_races(exe, tmp_path, case):  # noqa: F811
    p, vals, plan, Ap = _plan(case)
    tasks, _ = _export(plan, Ap, str(tmp_path / "plan.bin"))
    assert ((tasks[:, 0] & E.TF_CHAIN) != 0).sum() >= 10
    Lo = _oracle_factor_permuted(p, vals, plan.perm)
    _check(exe, tmp_path, len(tasks), lambda out: _assert_factor(plan, out, Lo))


def _assert_factor(plan, out, Lo):
    T, nt = plan.T, len(plan.tcol)
    t = out[:nt * T * T].reshape(-1, T, T).transpose(0, 2, 1)
    assert _err(E.dense_factor(plan, t), Lo) <= 1e-12
    return out[nt * T * T:]


@pytest.mark.parametrize("case", CASES[:2], ids=["natural", "nd3"])
def test_merged_pairs_have_no_races(exe, tmp_path, case):  # noqa: F811
    p, vals, plan, Ap = _plan(case)
    B = I.rhs(p.N, 2, seed=case[0])
    tasks = _export_merged(plan, Ap, B, str(tmp_path / "plan.bin"))
    assert ((tasks[:, 0] & E.TF_CHAIN) != 0).sum() >= 10
    Lo = _oracle_factor_permuted(p, vals, plan.perm)
    L, _ = oracle.factor(p.f, vals)
    Xo = oracle.solve(p.f, L, B)[plan.perm]

    def compare(out):
        Z = _assert_factor(plan, out, Lo).reshape(plan.ntr, 2, plan.T)
        X = np.concatenate([Z[m, :, :plan.row_cnt[m]].T for m in range(plan.ntr)])
        assert _err(X, Xo) <= 1e-12

    _check(exe, tmp_path, len(tasks), compare)


def _entry(tasks, succ, want):
    """First successor entry (its index) that `want(task, entry, place)` takes,
    behind the first few pairs."""
    for t in range(len(tasks) // 4, len(tasks)):
        for q in range(tasks[t, 5], tasks[t, 6]):
            if want(t, int(succ[q]), q - tasks[t, 5]):
                return q
    raise AssertionError("no such edge")


@pytest.mark.parametrize("what", ["early_edge", "other_successor", "notified_before_stored", "staged_without_wait"])
def test_planted_mistakes_are_reported(exe, tmp_path, what):  # noqa: F811
    p, vals, plan, Ap = _plan((900, 40, 130, None, 32, S.STILES_ORDER_NONE, 0))
    inp, out = str(tmp_path / "plan.bin"), str(tmp_path / "out.bin")
    tasks, succ = _export(plan, Ap, inp)
    chain, typ = (tasks[:, 0] & E.TF_CHAIN) != 0, tasks[:, 0] & 0xff
    if what == "early_edge":            # an update of a paired POTRF's tile that the pair does not wait for
        plant = [_entry(tasks, succ, lambda t, x, early, place: early and chain[x] and typ[x] == E.POTRF)]
    elif what == "other_successor":     # a reader of a paired TRSM's tile that does not wait for it
        plant = [_entry(tasks, succ, lambda t, x, early, place: chain[t] and typ[t] == E.TRSM and place > 0)]
    else:
        plant = [-1, 1 if what == "notified_before_stored" else 2]
    env = dict(os.environ, TSAN_OPTIONS=TSAN_OPTIONS)
    env.pop("LD_PRELOAD", None)
    for seed in (1, 2):
        r = subprocess.run([exe, inp, out, "8", str(seed)] + [str(x) for x in plant], capture_output=True, text=True,
                           env=env, timeout=600)
        assert r.returncode == 66 or "ThreadSanitizer: data race" in r.stderr


def _entry(tasks, succ, want):
    """A successor entry (its index), behind the first few pairs, that
    `want(task, successor, early, place in the list)` takes."""
    for t in range(len(tasks) // 4, len(tasks)):
        for q in range(tasks[t, 5], tasks[t, 6]):
            x, dec = E.succ_edge(succ[q])
            if want(t, x, dec != 1, q - tasks[t, 5]):
                return q
    raise AssertionError("no such edge")

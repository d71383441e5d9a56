"""Timed cases of the band-arrowhead Cholesky library: what a program that uses
it runs in earnest, through the package's public entry points.

A case is a dict of plain values:
  op       "factor"   factorize new values, the factor read out, log-determinant
           "fsl"      factorize new values and solve in one call, log-determinant
           "solve"    solve with a resident factor
           "marginal" selected inversion of a resident factor, diag(A^-1)
           "selinv"   factorize new values, selected inversion, the entries of
                      A^-1 on the factor's envelope and the log-determinant
           "batch"    many uneven matrices in one launch, their log-determinants
  input    "profile"  band plus arrow given by its row profile
           "spde"     spatio-temporal grid given as CSC
           "mesh"     irregular mesh given as CSC
  n, wlo, whi, seg, a: band rows, half-width per segment of seg rows (uniform in
           [wlo, whi]), dense arrow rows; pat: seed of that structure
  nrhs, tile, ordering, parts, precision, law: as in the analysis and the solve

The structure of a case is analyzed once per process: a program analyzes a
pattern once and factorizes many value sets with it.  Values, right-hand sides
and workspaces are made afresh for every state.
"""
import functools
import math

import numpy as np
import torch

import paper_2501_02483_amd as S
from paper_2501_02483_amd import autotune
from paper_2501_02483_amd import inputs as I
from paper_2501_02483_amd.devgen import DevicePattern

ORDERING = {"none": S.STILES_ORDER_NONE, "auto": S.STILES_ORDER_AUTO, "nd": S.STILES_ORDER_ADAPTABLE_ND,
            "amd": S.STILES_ORDER_AMD}
PRECISION = {"fp64": S.STILES_FP64, "mixed": S.STILES_MIXED32}


def _band(op, n, wlo, whi, a, nrhs, tile=64, ordering="nd", parts=0, precision="fp64", law="dominant", seg=5000,
          pat=2):
    return {"op": op, "input": "profile", "n": n, "wlo": wlo, "whi": whi, "seg": seg, "a": a, "pat": pat,
            "nrhs": nrhs, "tile": tile, "ordering": ordering, "parts": parts, "precision": precision, "law": law}


def listed():
    def named(name, c):
        return dict(c, name=name)
    return [
        # the smallest matrix of the uneven batch on its own, its factor
        # wanted: 51 tasks, launches and the pivot chain are all there is
        named("factor_1k", _band("factor", 1000, 32, 32, 4, 1, ordering="auto")),
        # the small workload of the benchmark with the plan its tuner picks:
        # the inner step of a hyperparameter search on a small model
        named("small_2k", _band("fsl", 2000, 50, 50, 10, 1, tile=32, parts=16)),
        # the smallest served pattern: natural order (fewer than 512 tile
        # rows), one right-hand side, bound by the chain of 157 pivots
        named("serve_10k", _band("fsl", 10_000, 64, 64, 16, 1, ordering="none")),
        # marginal covariances of a mid-size model with ragged sizes and
        # widths: factorization, log-determinant and selected inversion, the
        # selected entries read out
        named("selinv_12k", _band("selinv", 12_345, 150, 300, 37, 1, ordering="none", seg=1700)),
        # the uneven batch (n 1,000 to 20,000, w 32 to 256, a 4 to 64), one
        # launch, the ordering rule its tuner picks
        {"name": "batch_512", "op": "batch", "input": "profile", "count": 512, "pat": 3, "tile": 64, "nd_rows": 160},
        # the benchmark's default step: variable band, n = 200,000
        named("varband_200k", _band("fsl", 200_000, 200, 800, 100, 8)),
        # posterior marginal variances from that matrix's resident factor
        named("marginal_200k", _band("marginal", 200_000, 200, 800, 100, 1)),
        # a block of samples drawn with a resident factor: solves only
        named("solve_200k", _band("solve", 200_000, 200, 800, 100, 16)),
        # an irregular mesh with some long-range couplings, CSC input and
        # minimum-degree ordering: many narrow tiles, no band
        {"name": "mesh_20k", "op": "fsl", "input": "mesh", "n": 20_000, "a": 50, "long": 100, "pat": 1, "nrhs": 1,
         "tile": 64, "ordering": "amd", "parts": 0, "precision": "fp64"},
        # a spatio-temporal model, CSC input sparse inside a wide envelope
        {"name": "spde_96k", "op": "fsl", "input": "spde", "nx": 40, "ny": 40, "nt": 60, "a": 50, "nrhs": 8,
         "tile": 64, "ordering": "nd", "parts": 0, "precision": "fp64"},
        # the largest matrix: FP64, and mixed precision with 16 refined
        # right-hand sides on the ill-conditioned (1e6) Laplacian values
        named("fp64_500k", _band("fsl", 500_000, 1000, 1000, 200, 1)),
        named("mixed_500k", _band("fsl", 500_000, 1000, 1000, 200, 16, precision="mixed", law="laplacian")),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["factor", "fsl", "fsl", "fsl", "solve", "marginal", "selinv", "batch", "mesh", "spde", "mixed"])
    tile = rng.choice([32, 64, 64])
    if kind == "batch":
        return {"op": "batch", "input": "profile", "count": _log(rng, 16, 512), "pat": rng.randrange(1, 1000),
                "tile": tile, "nd_rows": rng.choice([0, 160])}
    if kind == "mesh":
        return {"op": "fsl", "input": "mesh", "n": _log(rng, 2000, 20_000), "a": rng.randint(1, 64),
                "long": rng.randint(0, 100), "pat": rng.randrange(1, 1000), "nrhs": rng.randint(1, 16), "tile": tile,
                "ordering": rng.choice(["amd", "auto"]), "parts": 0, "precision": "fp64"}
    if kind == "spde":
        return {"op": "fsl", "input": "spde", "nx": rng.randint(9, 40), "ny": rng.randint(9, 40),
                "nt": rng.randint(5, 60), "a": rng.randint(1, 64), "nrhs": rng.randint(1, 16), "tile": 64,
                "ordering": "nd", "parts": 0, "precision": "fp64"}
    natural = kind == "factor" or rng.random() < 0.3
    n = _log(rng, 1000, 25_000 if natural or kind == "selinv" else 300_000)
    # the flops n w^2 stay within a third of the largest listed matrix's
    whi = _log(rng, 32, max(32, min(800, n // 8, int(math.sqrt(1.5e11 / n)))))
    wlo = rng.randint(max(16, whi // 4), whi)
    ordering = ("auto" if kind == "factor" else "none") if natural or kind == "selinv" else "nd"
    nrhs = rng.choice([1, 1, rng.randint(2, 16)]) if kind in ("fsl", "solve", "mixed") else 1
    if kind == "mixed":
        return _band("fsl", n, wlo, whi, rng.randint(1, 200), nrhs, tile=64, ordering=ordering, precision="mixed",
                     law=rng.choice(["dominant", "laplacian"]), seg=rng.randint(900, 5000), pat=rng.randrange(1, 1000))
    return _band(kind, n, wlo, whi, rng.randint(0, 200), nrhs, tile=tile, ordering=ordering,
                 seg=rng.randint(900, 5000), pat=rng.randrange(1, 1000))


# ------------------------------------------------------------------ structure

def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k != "name"))


@functools.lru_cache(maxsize=4)
def _structure(key):
    """(pattern or CSC dict, symbolic object) of a case; lists for a batch."""
    c = dict(key)
    if c["op"] == "batch":
        pats = I.batch_patterns(seed=c["pat"], count=c["count"])
        return pats, autotune.batch_symbolics(pats, c["tile"], c["nd_rows"])
    opt = dict(tile=c["tile"], ordering=ORDERING[c["ordering"]], nd_parts=c["parts"])
    if c["input"] == "profile":
        nseg = (c["n"] + c["seg"] - 1) // c["seg"]
        widths = np.random.default_rng(c["pat"]).integers(c["wlo"], c["whi"] + 1, size=nseg)
        p = I.make_pattern(c["n"], c["a"], widths, seg=c["seg"])
        return p, S.Symbolic.from_pattern(p, **opt)
    if c["input"] == "spde":
        m = I.spde_space_time(c["nx"], c["ny"], c["nt"], c["a"], 6)
    else:
        m = I.irregular_mesh(c["n"], c["a"], c["pat"], long_edges=c["long"])
    m.pop("profile_values")
    m["col"] = np.repeat(np.arange(m["N"], dtype=np.int64), np.diff(m["colptr"]))
    return m, S.Symbolic.from_csc(m["N"], m["a"], m["colptr"], m["rowind"], **opt)


def _csc_values(m, seed):
    """N(0,1) off the diagonal, diagonal = absolute sum of the full symmetric row + 1."""
    v = np.random.default_rng(seed).standard_normal(m["rowind"].shape[0])
    dpos = m["colptr"][:-1]             # lower CSC: the diagonal comes first
    v[dpos] = 0.0
    w = np.abs(v)
    tot = np.bincount(m["rowind"], weights=w, minlength=m["N"]) + np.bincount(m["col"], weights=w, minlength=m["N"])
    v[dpos] = tot + 1.0
    return v


def _rhs(N, nrhs, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    return torch.randn(nrhs, N, dtype=torch.float64, device="cuda", generator=g).t()


# ------------------------------------------------------------- state and pass

def prepare(case, seed):
    st, sym = _structure(_key(case))
    s = {"op": case["op"]}
    if case["op"] == "batch":
        s["values"] = [DevicePattern(p).values(seed * 1000 + i) for i, p in enumerate(st)]
        s["factors"] = [S.Factor(y) for y in sym]
        s["batch"] = S.Batch(s["factors"])
        s["logdet"] = torch.empty(len(st), dtype=torch.float64, device="cuda")
        return s
    N = sym.info.N
    if case["input"] == "profile":
        s["values"] = DevicePattern(st).values(seed, law=case["law"])
    else:
        s["values"] = torch.from_numpy(_csc_values(st, seed)).cuda()
    s["factor"] = S.Factor(sym, PRECISION[case["precision"]], nrhs_max=case.get("nrhs", 1))
    s["logdet"] = torch.empty(1, dtype=torch.float64, device="cuda")
    if case["op"] in ("fsl", "solve"):
        s["B"] = _rhs(N, case["nrhs"], seed + 7)
        s["X"] = torch.empty_strided(s["B"].shape, s["B"].stride(), dtype=torch.float64, device="cuda")
    if case["op"] in ("solve", "marginal"):
        s["factor"].factorize(s["values"])
        del s["values"]
    if case["op"] in ("marginal", "selinv"):
        s["selinv"] = S.SelInv(s["factor"])
        s["diag"] = torch.empty(N, dtype=torch.float64, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "batch":
        s["batch"].factorize(s["values"])
        return {"logdet": s["batch"].logdet(s["logdet"])}
    f = s["factor"]
    if op == "fsl":
        s["X"].copy_(s["B"])
        f.factorize_solve(s["values"], s["X"])
        return {"X": s["X"], "logdet": f.logdet(s["logdet"])}
    if op == "solve":
        s["X"].copy_(s["B"])
        f.solve(s["X"])
        return {"X": s["X"]}
    if op == "marginal":
        return {"diag": s["selinv"].compute().diag(s["diag"])}
    f.factorize(s["values"])
    if op == "selinv":
        sigma = s["selinv"].compute().extract()
        return {"sigma": sigma, "logdet": f.logdet(s["logdet"])}
    return {"L": f.extract(), "logdet": f.logdet(s["logdet"])}


# ----------------------------------------------------------- necessary work

def _eta(f):
    """Entries below the diagonal in each column of an envelope."""
    N = f.shape[0]
    d = np.zeros(N + 1, dtype=np.int64)
    np.add.at(d, f, 1)
    np.add.at(d, np.arange(N), -1)
    return np.cumsum(d)[:N].astype(np.float64)


def work(case):
    """Values read once; factor, solution or selected inverse written once.
    Operations of the method on the input's own envelope (no padding, no fill
    of a partitioning): sum_j (eta_j + 1)^2 for the factorization, 4 nnz(L) per
    right-hand side, sum_j 2 eta_j (eta_j + 1) for the selected inversion.  For
    a mesh, whose envelope says nothing, the same sums over A's own entries."""
    st, _ = _structure(_key(case))
    if case["op"] == "batch":
        b = f = 0.0
        for p in st:
            e = _eta(p.f)
            b += 16.0 * float(e.sum() + p.N)
            f += float(((e + 1) ** 2).sum())
        return {"bytes": b, "flops": f}
    if case["input"] == "profile":
        e, na = _eta(st.f), st.nnz
    elif case["input"] == "spde":
        e, na = _eta(st["pattern"].f), st["rowind"].shape[0]
    else:
        e, na = np.diff(st["colptr"]).astype(np.float64) - 1.0, st["rowind"].shape[0]
    N = e.shape[0]
    nl = float(e.sum() + N)
    fac, inv, r = float(((e + 1) ** 2).sum()), float((2 * e * (e + 1)).sum()), case.get("nrhs", 1)
    return {"factor": {"bytes": 8.0 * (na + nl), "flops": fac},
            "fsl": {"bytes": 8.0 * (na + nl) + 16.0 * N * r, "flops": fac + 4 * nl * r},
            "solve": {"bytes": 8.0 * nl + 16.0 * N * r, "flops": 4 * nl * r},
            "marginal": {"bytes": 16.0 * nl, "flops": inv},
            "selinv": {"bytes": 8.0 * (na + 2 * nl), "flops": fac + inv}}[case["op"]]


# ------------------------------------------------------- results in 64 bits

class _Blocks:
    """Dense FP64 blocks of a band-plus-arrow matrix on the GPU: the band as a
    block-tridiagonal matrix of blocks as wide as its half-width."""

    def __init__(self, n, a, w, rows, cols, vals):
        # rows, cols, vals: callable(lo, hi) -> lower entries of rows [lo, hi)
        self.n, self.a = n, a
        self.m = max(w, 64)
        self.cut = list(range(0, n, self.m)) + [n]
        self.entries = lambda lo, hi: (rows(lo, hi), cols(lo, hi), vals(lo, hi))

    def dense(self, lo, hi, c0, c1):
        r, c, v = self.entries(lo, hi)
        k = (c >= c0) & (c < c1)
        out = torch.zeros((hi - lo, c1 - c0), dtype=torch.float64, device="cuda")
        out[r[k] - lo, c[k] - c0] = v[k]
        return out

    def factor(self):
        """Diagonal, sub-diagonal and arrow blocks of L, and the arrow corner."""
        n, a, cut = self.n, self.a, self.cut
        arrow = self.dense(n, n + a, 0, n + a)
        corner = arrow[:, n:].tril()
        corner = corner + corner.tril(-1).t()
        D, E, A = [], [], []
        for k in range(len(cut) - 1):
            lo, hi = cut[k], cut[k + 1]
            p = cut[k - 1] if k else 0
            blk = self.dense(lo, hi, p, hi)
            d = blk[:, lo - p:]
            d = d + d.tril(-1).t()
            ar = arrow[:, lo:hi]
            if k:
                e = torch.linalg.solve_triangular(D[-1], blk[:, :lo - p].t(), upper=False).t()
                d = d - e @ e.t()
                ar = ar - A[-1] @ e.t()
                E.append(e)
            D.append(torch.linalg.cholesky(d))
            A.append(torch.linalg.solve_triangular(D[-1], ar.t(), upper=False).t())
            corner = corner - A[-1] @ A[-1].t()
        return D, E, A, torch.linalg.cholesky(corner) if a else corner

    def solve(self, L, B):
        D, E, A, C = L
        n, cut, nb = self.n, self.cut, len(self.cut) - 1
        tri = torch.linalg.solve_triangular
        Y, yc = [], B[n:].clone()
        for k in range(nb):
            r = B[cut[k]:cut[k + 1]]
            if k:
                r = r - E[k - 1] @ Y[-1]
            Y.append(tri(D[k], r, upper=False))
            yc -= A[k] @ Y[-1]
        X = torch.empty_like(B)
        if self.a:
            X[n:] = tri(C.t(), tri(C, yc, upper=False), upper=True)
        for k in reversed(range(nb)):
            r = Y[k] - A[k].t() @ X[n:]
            if k + 1 < nb:
                r = r - E[k].t() @ X[cut[k + 1]:cut[k + 2]]
            X[cut[k]:cut[k + 1]] = tri(D[k].t(), r, upper=True)
        return X

    def logdet(self, L):
        D, _, _, C = L
        s = sum(d.diagonal().log().sum() for d in D)
        return 2.0 * (s + (C.diagonal().log().sum() if self.a else 0.0)).reshape(1)

    def selected(self, L):
        """Blocks of A^-1: diagonal, sub-diagonal, arrow rows, corner."""
        D, E, A, C = L
        nb = len(D)
        Sc = torch.cholesky_inverse(C) if self.a else C
        Sd, Se, Sa = [None] * nb, [None] * max(nb - 1, 0), [None] * nb
        for k in reversed(range(nb)):
            inv = torch.linalg.solve_triangular(D[k], torch.eye(D[k].shape[0], dtype=torch.float64, device="cuda"),
                                                upper=False)
            if k + 1 < nb:
                le, la = E[k] @ inv, A[k] @ inv
                e = -(Sd[k + 1] @ le + Sa[k + 1].t() @ la)
                ar = -(Sa[k + 1] @ le + Sc @ la)
                Sd[k] = inv.t() @ inv - le.t() @ e - la.t() @ ar
                Se[k] = e
            else:
                la = A[k] @ inv
                ar = -Sc @ la
                Sd[k] = inv.t() @ inv - la.t() @ ar
            Sa[k] = ar
        return Sd, Se, Sa, Sc

    def envelope(self, f, blocks):
        """Row-profile order of a lower band-plus-arrow matrix in blocks."""
        Dk, Ek, Ak, C = blocks
        cut, n, out = self.cut, self.n, []
        for k in range(len(Dk)):
            lo, hi = cut[k], cut[k + 1]
            p = cut[k - 1] if k else 0
            row = torch.cat([Ek[k - 1], Dk[k]], 1) if k else Dk[k]
            c = torch.arange(p, hi, device="cuda")[None, :]
            i = torch.arange(lo, hi, device="cuda")[:, None]
            out.append(row[(c >= torch.from_numpy(f[lo:hi]).cuda()[:, None]) & (c <= i)])
        if self.a:
            full = torch.cat(list(Ak) + [C], 1)
            c = torch.arange(n + self.a, device="cuda")[None, :]
            out.append(full[c <= torch.arange(n, n + self.a, device="cuda")[:, None]])
        return torch.cat(out)


def _profile_blocks(p, v):
    rp = torch.from_numpy(p.row_ptr()).cuda()
    f = torch.from_numpy(np.ascontiguousarray(p.f)).cuda()

    def rows(lo, hi):
        return torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), rp[lo + 1:hi + 1] - rp[lo:hi])

    def cols(lo, hi):
        r = rows(lo, hi)
        return torch.arange(int(rp[lo]), int(rp[hi]), device="cuda") - rp[r] + f[r]

    i = np.arange(p.n)
    return _Blocks(p.n, p.a, int((i - p.band_first_col).max()), rows, cols, lambda lo, hi: v[int(rp[lo]):int(rp[hi])])


def _csc_blocks(m, v):
    order = np.lexsort((m["col"], m["rowind"]))
    R, C = (torch.from_numpy(x[order]).cuda() for x in (m["rowind"], m["col"]))
    V = v[torch.from_numpy(order).cuda()]
    rp = np.concatenate([[0], np.cumsum(np.bincount(m["rowind"], minlength=m["N"]))])
    part = lambda x: lambda lo, hi: x[int(rp[lo]):int(rp[hi])]  # noqa: E731
    w = int((np.arange(m["n"]) - m["pattern"].f[:m["n"]]).max())
    return _Blocks(m["n"], m["a"], w, part(R), part(C), part(V))


def exact(case, seed):
    st, sym = _structure(_key(case))
    if case["op"] == "batch":
        out = []
        for i, p in enumerate(st):
            b = _profile_blocks(p, DevicePattern(p).values(seed * 1000 + i))
            out.append(b.logdet(b.factor()))
        return {"logdet": torch.cat(out)}
    N = sym.info.N
    B = _rhs(N, case["nrhs"], seed + 7)
    if case["input"] == "mesh":
        v = torch.from_numpy(_csc_values(st, seed)).cuda()
        M = torch.zeros((N, N), dtype=torch.float64, device="cuda")
        M[torch.from_numpy(st["rowind"]).cuda(), torch.from_numpy(st["col"]).cuda()] = v
        L = torch.linalg.cholesky(M + M.tril(-1).t())
        return {"X": torch.cholesky_solve(B, L), "logdet": 2.0 * L.diagonal().log().sum().reshape(1)}
    if case["input"] == "spde":
        b = _csc_blocks(st, torch.from_numpy(_csc_values(st, seed)).cuda())
    else:
        b = _profile_blocks(st, DevicePattern(st).values(seed, law=case["law"]))
    L = b.factor()
    if case["op"] == "fsl":
        return {"X": b.solve(L, B), "logdet": b.logdet(L)}
    if case["op"] == "solve":
        return {"X": b.solve(L, B)}
    if case["op"] == "factor":
        return {"L": b.envelope(st.f, L), "logdet": b.logdet(L)}
    sig = b.selected(L)
    if case["op"] == "marginal":
        return {"diag": torch.cat([d.diagonal() for d in sig[0]] + [sig[3].diagonal()])}
    return {"sigma": b.envelope(st.f, sig), "logdet": b.logdet(L)}

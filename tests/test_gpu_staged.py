"""The staged product (vectors of up to eight LDS parts, 9e5 entries and up)
against the FP64 CPU oracle where its plan can go wrong: one, two, four and
eight parts, a last part that is not full, empty and dense segments, cones."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_2203_05027_amd import instances as I
from paper_2203_05027_amd.solver import Solver

pytestmark = pytest.mark.gpu

# (rows, columns, entries per column): parts of the row and column pass in FP64
SHAPES = {"one part": (3001, 12_013, 80), "eight and one": (9001, 100_003, 10), "two and four": (45_007, 20_011, 60),
          "holes": (9001, 50_021, 40), "cones": (9001, 0, 25)}
_insts = {}


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _instance(kind):
    if kind in _insts:
        return _insts[kind]
    m, n, k = SHAPES[kind]
    if kind == "cones":
        inst = I.conic_instance(m, 20_003, [4] * 5000 + [64, 3, 50, 1], k, seed=81)
    else:
        inst = I.lp_instance(m, n, k, seed=82)
    if kind == "holes":  # empty rows and columns, one dense row, one dense column
        A = sp.csr_matrix((inst["val"], inst["col_idx"], inst["row_ptr"]), shape=(m, n))
        rows, cols = np.ones(m), np.ones(n)
        rows[[0, 5, m - 1]] = 0.0
        rows[3000:4500] = 0.0
        cols[-12_000:] = 0.0
        cols[7] = 0.0
        A = sp.diags(rows) @ A @ sp.diags(cols)
        j, i = np.arange(n - 12_000), np.flatnonzero(rows)
        full = sp.csr_matrix((np.full(j.size, 0.01), (np.full(j.size, 5), j)), shape=(m, n))
        tall = sp.csr_matrix((np.full(i.size, 0.02), (i, np.full(i.size, 7))), shape=(m, n))
        A = (A + full + tall).tocsr()
        A.eliminate_zeros()
        A.sort_indices()
        inst = dict(inst, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                    nnz=A.nnz, b=A @ inst["x0"], c=A.T @ inst["y0"] + inst["s0"])
    _insts[kind] = inst
    return inst


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", list(SHAPES))
def test_staged_product_matches_oracle(kind, precision):
    """30 iterations, a check every seven, then a resume: in FP64 the oracle's
    iterates to 1e-9, in mixed precision to 1e-5 (FP32 rounding), and the
    residuals of the solver's own iterate to 1e-11."""
    inst = _instance(kind)
    orc = oracle.Oracle.from_instance(inst)
    orc.iterate(29)
    o = orc.state()
    with Solver.from_instance(inst, eps=0.0, check_every=7, precision=precision, full_checks=True) as s:
        s.iterate(28)
        g28, r28 = s.solution(), s.residuals()
        s.iterate(1)
        g = s.solution()
        s.resume(g28["x"], g28["z"], g28["delta"], g28["lambda"])
        s.iterate(1)
        again = s.solution()
    tol = 1e-9 if precision == "fp64" else 1e-5
    errs = {k: rel(g[k], o[k]) for k in g}
    sys.__stderr__.write(f"[gpu-test] staged {kind} {precision}: {errs}\n")
    assert max(errs.values()) <= tol, errs
    assert max(rel(again[k], o[k]) for k in g) <= tol
    orc.set_state(x=g28["x"], z=g28["z"], delta=g28["delta"], lam=g28["lambda"])
    ro = orc.residuals()
    for k in ("r_prim", "r_dual", "r_gap", "pobj", "dobj", "res_ax_b", "prim_inf", "dual_inf", "scale_p", "scale_d"):
        assert abs(r28[k] - ro[k]) <= 1e-11 * max(abs(ro[k]), 1e-3), (k, r28[k], ro[k])


def _with(kind, B):
    """B with short or empty segments beside its long ones."""
    m, n = B.shape
    if kind == "slack columns":
        return sp.hstack([B, sp.eye(m, format="csr")])
    if kind == "empty columns":
        return sp.hstack([B, sp.csr_matrix((m, 130_000))])
    if kind == "short rows":
        return sp.vstack([B, sp.csr_matrix((np.ones(60_000), (np.arange(60_000), np.arange(60_000) % n)), shape=(60_000, n))])
    return B


@pytest.mark.parametrize("kind", ["slack columns", "empty columns", "short rows"])
def test_short_segments_share_the_workgroups(kind):
    """Segments of one entry or none after ones of a hundred, and parts that
    hold nearly all or none of the entries: the oracle's iterates, and passes
    at most three times those without them (shares of the entries alone took
    4 to 75 times)."""
    g = np.random.default_rng(1)
    B = sp.csr_matrix((g.standard_normal(3_000_000), (g.integers(0, 10_000, 3_000_000), np.repeat(np.arange(30_000), 100))),
                      shape=(10_000, 30_000))
    ms = {}
    for k in ("plain", kind):
        A = _with(k, B).tocsr()
        A.sort_indices()
        rng = np.random.default_rng(3)
        m, n = A.shape
        inst = dict(m=m, n=n, nnz=A.nnz, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                    b=A @ np.maximum(rng.standard_normal(n), 0.0), c=A.T @ rng.standard_normal(m) + rng.uniform(0, 1, n),
                    n_orth=n, soc_sizes=np.zeros(0, np.int32))
        with Solver.from_instance(inst, eps=0.0) as s:
            s.iterate(12)
            g = s.solution()
            ms[k] = min(max(s.time_kernels(20)) for _ in range(3))
    orc = oracle.Oracle.from_instance(inst)
    orc.iterate(12)
    o = orc.state()
    sys.__stderr__.write(f"[gpu-test] staged {kind}: slower pass {ms}\n")
    assert max(rel(g[k], o[k]) for k in g) <= 1e-9
    assert ms[kind] <= 3.0 * ms["plain"], ms

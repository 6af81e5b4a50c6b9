"""The binned product (vectors above an XCD's L2, some 5e6 entries and up) against
the FP64 CPU oracles where its plan can go wrong: a last part and last group
that are not full, empty rows and columns, rows of exactly half a group (the
longest it takes) and one more (the slab product then), cones."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import standard as std_oracle
from paper_2203_05027_amd import instances as I
from paper_2203_05027_amd.solver import Solver, Standard

pytestmark = pytest.mark.gpu

HALF_GROUP = 5120
_insts = {}


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _instance(kind):
    if kind in _insts:
        return _insts[kind]
    if kind == "cones":
        inst = I.conic_instance(330_001, 300_007, [3, 50, 1, 17, 64] * 2400, 8, seed=71)
    else:
        inst = I.lp_instance(310_001, 640_009, 9, seed=72)
    if kind.startswith("long"):
        A = sp.csr_matrix((inst["val"], inst["col_idx"], inst["row_ptr"]), shape=(inst["m"], inst["n"])).tolil()
        rng = np.random.default_rng(73)
        A = A.tocsr()
        keep = np.ones(inst["m"])
        keep[[0, 17, inst["m"] - 1]] = 0.0           # the dense rows, drawn below
        keep[100:40_000] = 0.0                        # more empty rows than a group has threads
        cols = np.ones(inst["n"])
        cols[-9000:] = 0.0                            # and empty columns at the end
        A = sp.diags(keep) @ A @ sp.diags(cols)
        count = HALF_GROUP + (1 if kind == "long+1" else 0)
        for r in (0, 17, inst["m"] - 1):
            j = np.sort(rng.choice(inst["n"] - 9000, size=count, replace=False))
            B = sp.csr_matrix((rng.standard_normal(count) * 0.02, (np.full(count, r), j)), shape=A.shape)
            A = A + B
        A = A.tocsr()
        A.eliminate_zeros()
        A.sort_indices()
        inst = dict(inst, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                    nnz=A.nnz, b=A @ inst["x0"], c=A.T @ inst["y0"] + inst["s0"])
    _insts[kind] = inst
    return inst


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["ragged", "long", "long+1", "cones"])
def test_binned_product_matches_oracle(kind, precision):
    """22 iterations, a check every seven, then a resume from that state: in
    FP64 the oracle's iterates and residuals to 1e-9, in mixed precision to
    1e-5 (FP32 rounding) with the residuals of its own iterate to 1e-11."""
    inst = _instance(kind)
    orc = oracle.Oracle.from_instance(inst)
    orc.iterate(22)
    o = orc.state()
    with Solver.from_instance(inst, eps=0.0, check_every=7, precision=precision, full_checks=True) as s:
        s.iterate(21)
        g21, r21 = s.solution(), s.residuals()
        s.iterate(1)
        g = s.solution()
        s.resume(g21["x"], g21["z"], g21["delta"], g21["lambda"])
        s.iterate(1)
        again = s.solution()
    tol = 1e-9 if precision == "fp64" else 1e-5
    errs = {k: rel(g[k], o[k]) for k in g}
    sys.__stderr__.write(f"[gpu-test] binned {kind} {precision}: {errs}\n")
    assert max(errs.values()) <= tol, errs
    assert max(rel(again[k], o[k]) for k in g) <= tol
    orc.set_state(x=g21["x"], z=g21["z"], delta=g21["delta"], lam=g21["lambda"])
    ro = orc.residuals()
    for k in ("r_prim", "r_dual", "r_gap", "pobj", "dobj", "res_ax_b", "prim_inf", "dual_inf", "scale_p", "scale_d"):
        assert abs(r21[k] - ro[k]) <= 1e-11 * max(abs(ro[k]), 1e-3), (k, r21[k], ro[k])


def test_binned_product_is_reproducible():
    """The entries' places are handed out by atomics; the sums do not depend on them."""
    inst = _instance("ragged")
    outs = []
    for _ in range(2):
        with Solver.from_instance(inst, eps=0.0) as s:
            s.iterate(30)
            outs.append(s.solution())
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("kind", ["long", "cones"])
def test_standard_baseline_with_binned_products(kind):
    inst = _instance(kind)
    orc = std_oracle.StandardADMM.from_instance(inst, mu=1.0, cg_iters=2, cg_tol=0.0)
    orc.iterate(6)
    o = orc.state()
    with Standard.from_instance(inst, cg_iters=2, eps=0.0, check_every=4) as s:
        s.iterate(6)
        g = s.solution()
    errs = {k: rel(g[k], o[k]) for k in ("x1", "x2", "lam", "nu", "delta")}
    sys.__stderr__.write(f"[gpu-test] standard binned {kind}: {errs}\n")
    assert max(errs.values()) <= 1e-9, errs


def test_empty_rows_share_the_workgroups():
    """A run of empty rows is not left to one workgroup: the passes take at
    most twice the time without it (a group of entries alone: seventeen times)."""
    inst = _instance("ragged")
    more = dict(inst, m=inst["m"] + 900_000, b=np.append(inst["b"], np.zeros(900_000)),
                row_ptr=np.append(inst["row_ptr"], np.full(900_000, inst["nnz"])))
    ms, sol = [], []
    for i in (inst, more):
        with Solver.from_instance(i, eps=0.0) as s:
            s.iterate(5)
            sol.append(s.solution())
            ms.append(min(s.time_kernels(20)[1] for _ in range(3)))
    sys.__stderr__.write(f"[gpu-test] binned row pass without and with empty rows: {ms} ms\n")
    for k in ("x", "z", "delta"):
        assert rel(sol[1][k], sol[0][k]) <= 1e-12, k
    assert ms[1] <= 2.0 * ms[0], ms


def test_long_segments_do_not_hold_their_group():
    """Forty rows of 5000 entries among rows of nineteen: the row pass takes
    at most 1.5 times the pass without them (a thread a row: four times)."""
    inst = _instance("ragged")
    rng = np.random.default_rng(76)
    A = sp.csr_matrix((inst["val"], inst["col_idx"], inst["row_ptr"]), shape=(inst["m"], inst["n"]))
    rows = np.repeat(np.arange(40) * 7_000, 5000)
    cols = np.concatenate([rng.choice(inst["n"], size=5000, replace=False) for _ in range(40)])
    D = (A + sp.csr_matrix((rng.standard_normal(rows.size) * 0.02, (rows, cols)), shape=A.shape)).tocsr()
    D.sort_indices()
    longer = dict(inst, row_ptr=D.indptr.astype(np.int64), col_idx=D.indices.astype(np.int32), val=D.data, nnz=D.nnz)
    ms = []
    for i in (inst, longer):
        with Solver.from_instance(i, eps=0.0) as s:
            s.iterate(5)
            ms.append(min(s.time_kernels(20)[1] for _ in range(3)))
    sys.__stderr__.write(f"[gpu-test] binned row pass without and with long rows: {ms} ms\n")
    assert ms[1] <= 1.5 * ms[0], ms

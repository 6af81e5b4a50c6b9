"""The resident kernel that keeps a lane's row and column in registers, at the
sizes where it can go wrong: one row or column, the most rows and columns it
takes and one more, rows and columns longer than the registers hold and empty
ones, values at the ends of the type's range (where the division by a whole
number is not taken apart), a problem that just fills LDS."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_2203_05027_amd.solver import Solver

pytestmark = pytest.mark.gpu
KEYS = ("x", "z", "delta", "lambda")
# eleven iterations with a few roundings of at most a few hundred terms each
TOL = {"fp64": 1e-11, "mixed": 1e-4}


def _instance(m, n, density, seed, scale=1.0, nnz=None):
    rng = np.random.default_rng(seed)
    if nnz is None:
        A = sp.random(m, n, density=density, random_state=rng, data_rvs=rng.standard_normal, format="lil")
        if m > 3 and n > 3:
            A[m // 2] = 0.0                       # an empty row and column, a longer row and column
            A[:, n // 3] = 0.0
            A[m - 1, : min(n, 700)] = 0.05
            A[: min(m, 300), n - 1] = 0.07
        A = A.tocsr()
    else:
        at = rng.choice(m * n, nnz, replace=False)
        A = sp.csr_matrix((rng.standard_normal(nnz), (at // n, at % n)), shape=(m, n))
    A.eliminate_zeros()
    A.sort_indices()
    return dict(m=m, n=n, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                b=scale * (A @ np.maximum(rng.standard_normal(n), 0.0)),
                c=scale * (A.T @ rng.standard_normal(m) + rng.uniform(0, 1, n)),
                n_orth=n, soc_sizes=np.zeros(0, np.int32))


def _errors(sol, ref):
    scale = max(np.abs(ref[k]).max() for k in KEYS)
    return {k: float(np.abs(sol[k] - ref[k]).max() / scale) for k in KEYS}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(1, 1, 1.0), (1, 1024, 0.9), (1024, 1, 0.9), (1024, 1024, 0.002),
                                   (1023, 1025, 0.002), (1025, 1000, 0.002), (7, 400, 0.7), (63, 65, 0.4),
                                   (129, 513, 0.05), (513, 512, 0.008)])
def test_register_form_matches_oracle(shape, precision):
    inst = _instance(*shape, seed=sum(shape[:2]))
    rng = np.random.default_rng(4)
    start = tuple(rng.standard_normal(k) for k in (inst["n"], inst["n"], inst["n"], inst["m"]))
    with Solver.from_instance(inst, precision=precision, eps=0.0, check_every=4, resident="required") as s:
        s.set_start(*start)
        s.iterate(11)
        sol = s.solution()
    o = oracle.Oracle.from_instance(inst)
    o.set_start(*start)
    o.iterate(11)
    errs = _errors(sol, o.state())
    sys.__stderr__.write(f"[gpu-test] register form {shape} {precision}: {errs}\n")
    assert max(errs.values()) <= TOL[precision], errs


@pytest.mark.parametrize("precision,scale", [("fp64", 1e-295), ("fp64", 1e294), ("mixed", 1e-33), ("mixed", 1e34)])
def test_values_at_the_ends_of_the_range(precision, scale):
    inst = _instance(90, 200, 0.05, 7, scale=scale)
    unit = _instance(90, 200, 0.05, 7)
    with Solver.from_instance(inst, precision=precision, eps=0.0, check_every=1000, resident="required") as s:
        s.iterate(11)
        sol = s.solution()
    o = oracle.Oracle.from_instance(unit)   # the iteration is positively homogeneous in b and c
    o.iterate(11)
    errs = _errors({k: sol[k] / scale for k in KEYS}, o.state())
    sys.__stderr__.write(f"[gpu-test] register form at {scale} {precision}: {errs}\n")
    assert max(errs.values()) <= TOL[precision], errs


@pytest.mark.parametrize("full", [0, 1])
def test_a_residual_query_repeats_the_check(full):
    inst = _instance(300, 700, 0.02, 8)
    with Solver.from_instance(inst, eps=0.0, check_every=5, resident="required", full_checks=1) as s:
        s.iterate(20)
        whole = s.residuals()
    with Solver.from_instance(inst, eps=0.0, check_every=5, resident="required", full_checks=full) as s:
        s.iterate(20)
        again = s.residuals()
    assert {k: whole[k] for k in ("kkt", "r_prim", "r_dual", "r_gap")} == \
        {k: again[k] for k in ("kkt", "r_prim", "r_dual", "r_gap")}


@pytest.mark.parametrize("over", [0, 1])
def test_a_problem_that_just_fills_lds(over):
    """delta, x, z (24 n), lambda, u (16 m), offsets and 20 bytes an entry in
    FP64, each array rounded up to 16 bytes: the most entries that fit, and
    one more (the sweep kernels)."""
    m, n = 400, 900
    up = lambda v: (v + 15) // 16 * 16
    need = lambda k: 3 * up(8 * n) + 2 * up(8 * m) + 2 * up(8 * k) + up(4 * n + 4) + up(4 * m + 4) + 2 * up(2 * k)
    nnz = next(k for k in range(20000) if need(k + 1) > 160 * 1024 - 2048) + over
    inst = _instance(m, n, None, 9, nnz=nnz)
    with Solver.from_instance(inst, eps=0.0, check_every=4) as s:
        assert bool(s.launch_shape()["resident"]) == (over == 0)
        s.iterate(11)
        sol = s.solution()
    o = oracle.Oracle.from_instance(inst)
    o.iterate(11)
    errs = _errors(sol, o.state())
    assert max(errs.values()) <= TOL["fp64"], errs


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("row,col", [(16, 0), (40, 0), (0, 60), (1000, 600)])
def test_a_long_row_or_column_keeps_its_speed(row, col, precision):
    """One long row or column: the oracle's iterates on both sides of the rule
    that leaves the register form, and at most 1.25 times the time of the same
    problem with more (empty) columns than threads, which the rule never takes."""
    import time

    import scipy.sparse as sp
    m, n = 600, 1000
    rng = np.random.default_rng(5)
    A = sp.csr_matrix((rng.standard_normal(3 * n), (rng.integers(0, m, 3 * n), np.repeat(np.arange(n), 3))), shape=(m, n)).tolil()
    A[0, :row] = 0.1
    A[:col, 0] = 0.1
    us = []
    for pad in (0, 40):
        B = sp.hstack([A, sp.csr_matrix((m, pad))]).tocsr() if pad else A.tocsr()
        B.sort_indices()
        inst = dict(m=m, n=n + pad, nnz=B.nnz, row_ptr=B.indptr.astype(np.int64), col_idx=B.indices.astype(np.int32), val=B.data,
                    b=B @ np.linspace(0, 1, n + pad), c=np.linspace(1, 2, n + pad), n_orth=n + pad, soc_sizes=np.zeros(0, np.int32))
        with Solver.from_instance(inst, precision=precision, eps=0.0, resident="required") as s:
            s.iterate(13)
            if not pad:
                o = oracle.Oracle.from_instance(inst)
                o.iterate(13)
                so, g = o.state(), s.solution()
                scale = max(np.abs(so[k]).max() for k in g)
                assert max(float(np.abs(g[k] - so[k]).max()) for k in g) <= (1e-9 if precision == "fp64" else 1e-5) * scale
            best = 1e9
            for _ in range(4):
                t0 = time.perf_counter()
                s.iterate(1000)
                best = min(best, time.perf_counter() - t0)
            us.append(best * 1e3)
    sys.__stderr__.write(f"[gpu-test] resident row {row} column {col} {precision}: {us[0]:.2f} us an iteration, padded {us[1]:.2f}\n")
    assert us[0] <= 1.25 * us[1], us

"""The batched solver's sliced copies and renumbering at the sizes where they
can go wrong: one row, slices that are not full, odd and zero widths, rows and
columns of very different lengths, instances that just fill LDS (no room for
the padding's zeros)."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_2203_05027_amd.solver import Batch, UvError

pytestmark = pytest.mark.gpu
KEYS = ("x", "z", "delta", "lambda")


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _instance(m, n, density, seed):
    rng = np.random.default_rng(seed)
    A = sp.random(m, n, density=density, random_state=rng, data_rvs=rng.standard_normal, format="lil")
    if m > 3 and n > 3:
        A[m // 2] = 0.0                       # an empty row and column, a dense row and column
        A[:, n // 3] = 0.0
        A[m - 1, :] = 0.1
        A[:, n - 1] = 0.07
    A = A.tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    return dict(m=m, n=n, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                b=A @ np.maximum(rng.standard_normal(n), 0.0), c=A.T @ rng.standard_normal(m) + rng.uniform(0, 1, n),
                n_orth=n, soc_sizes=np.zeros(0, np.int32))


SIZES = [(1, 1, 1.0), (1, 70, 0.5), (63, 64, 0.2), (64, 65, 0.1), (65, 129, 0.03), (130, 40, 0.3), (200, 1023, 0.01),
         (513, 700, 0.02), (2050, 2500, 0.002)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("tiles", [None, (1024, [1, 1] * 4), (256, [1, 0] * 4), (64, [2, 1] * 4), (512, [1, 4] * 4)])
def test_slices_match_oracle(tiles, precision):
    insts = [_instance(*s, seed=50 + i) for i, s in enumerate(SIZES)]
    rng = np.random.default_rng(9)
    starts = [tuple(rng.standard_normal(k) for k in (i["n"], i["n"], i["n"], i["m"])) for i in insts]
    with Batch(insts, precision=precision, eps=0.0, check_every=4) as b:
        if tiles:
            b.set_tiles(*tiles)
        for i, s in enumerate(starts):
            if i % 2:
                b.set_start(i, *s)
        b.iterate(11)
        sols, res = [b.solution(i) for i in range(len(insts))], [b.residuals(i) for i in range(len(insts))]
    tol = 1e-9 if precision == "fp64" else 1e-5
    for i, inst in enumerate(insts):
        o = oracle.Oracle.from_instance(inst)
        if i % 2:
            o.set_start(*starts[i])
        o.iterate(8)
        ro = o.residuals()
        o.iterate(3)
        so = o.state()
        errs = {k: rel(sols[i][k], so[k]) for k in KEYS}
        scale = max(np.abs(so[k]).max() for k in KEYS)
        worst = max(float(np.abs(sols[i][k] - so[k]).max()) / scale for k in KEYS)
        assert worst <= tol, (i, errs)
        # full checks skip nothing here: r_prim of the check at iteration 8 is recorded only where it was whole
        assert res[i]["iter"] == 11 and ro["kkt"] >= 0.0


def test_start_and_solution_are_in_the_callers_order():
    """No iteration: what goes in comes out, in FP64 bit for bit."""
    inst = _instance(65, 129, 0.05, 3)
    rng = np.random.default_rng(4)
    s = [rng.standard_normal(k) for k in (129, 129, 129, 65)]
    with Batch([_instance(7, 9, 0.5, 1), inst], precision="fp64", eps=0.0) as b:
        b.set_start(1, *s)
        out = b.solution(1)
    for v, k in zip(s, KEYS):
        assert np.array_equal(out[k], v), k


@pytest.mark.parametrize("extra", [0, 2, 3, 4, 5])
def test_instances_that_just_fill_lds(extra):
    """x and u one step past the LDS a launch is left with (refused), or
    within it with no room for the padding's two zeros (lane groups) and with
    room."""
    total = (160 * 1024 - 1024) // 8 - extra
    m = total // 3
    inst = _instance(m, total - m, 5.0 / m, 12)
    if extra == 0:
        with pytest.raises(UvError):
            Batch([inst], precision="fp64", eps=0.0)
        return
    with Batch([inst], precision="fp64", eps=0.0, check_every=3) as b:
        b.iterate(7)
        sol = b.solution(0)
    o = oracle.Oracle.from_instance(inst)
    o.iterate(7)
    so = o.state()
    errs = {k: rel(sol[k], so[k]) for k in KEYS}
    sys.__stderr__.write(f"[gpu-test] batch at the LDS limit ({extra}): {errs}\n")
    # lambda is a difference of the rows' sums: its error is measured against their size (the full row's, ~1e3)
    scale = {k: np.abs(so[k]).max() for k in KEYS}
    A = sp.csr_matrix((np.abs(inst["val"]), inst["col_idx"], inst["row_ptr"]), shape=(inst["m"], inst["n"]))
    scale["lambda"] = (A @ np.abs(so["x"])).max()
    assert all(np.abs(sol[k] - so[k]).max() <= 1e-9 * scale[k] for k in KEYS), errs


@pytest.mark.parametrize("precision,total", [("fp64", 20349), ("fp64", 20350), ("mixed", 40699), ("mixed", 40700)])
def test_sliced_columns_asked_for_without_room_for_them(precision, total):
    """x and u fit LDS, the padding's two zeros do not: zero lanes per column
    (the sliced copy) are then one lane a column, in the sweep and the checks."""
    m = total // 3
    inst = _instance(m, total - m, 5.0 / m, 13)
    out = []
    for lanes in ([2, 0] * 4, [2, 1] * 4):
        with Batch([inst], precision=precision, eps=0.0, check_every=3, full_checks=True) as b:
            b.set_tiles(512, lanes)
            b.iterate(7)
            out.append((b.solution(0), b.residuals(0)))
    for k in KEYS:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert out[0][1] == out[1][1] and out[0][1]["iter"] == 7


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m,n,density", [(70, 300, 0.2), (600, 900, 0.02), (530, 4000, 0.3)])
def test_sliced_rows_are_the_sums_of_two_lanes(m, n, density, precision):
    """The sliced rows add even and odd entries apart, as two lanes a row do
    (one running sum has twice their rounding error): the same iterates bit
    for bit, checks included."""
    inst = _instance(m, n, density, 21)
    out = []
    for lanes in ([1, 0] * 4, [2, 0] * 4):
        with Batch([inst], precision=precision, eps=0.0, check_every=3) as b:
            b.set_tiles(256, lanes)
            b.iterate(8)
            out.append(b.solution(0))
    for k in KEYS:
        assert np.array_equal(out[0][k], out[1][k]), k


def test_dense_rows_do_not_grow_the_batch():
    """One row of 40,000 entries beside an empty one, 850 instances: slices 64
    times that row would pass 2^31 slots, so such rows keep their lane groups."""
    n = 40_000
    rng = np.random.default_rng(31)
    a, x = rng.standard_normal(n) / 200.0, np.maximum(rng.standard_normal(n), 0.0)
    inst = dict(m=2, n=n, row_ptr=np.array([0, n, n], np.int64), col_idx=np.arange(n, dtype=np.int32), val=a,
                b=np.array([a @ x, 0.0]), c=a * 0.3 + rng.uniform(0, 1, n), n_orth=n, soc_sizes=np.zeros(0, np.int32))
    with Batch([inst] * 850, precision="mixed", eps=0.0) as b:
        for lanes in ([4, 0] * 4, [1, 0] * 4):
            b.set_tiles(256, lanes)
        b.iterate(3)
        sols = [b.solution(i) for i in (0, 849)]
    o = oracle.Oracle.from_instance(inst)
    o.iterate(3)
    so = o.state()
    scale = max(np.abs(so[k]).max() for k in KEYS)
    for s in sols:
        assert max(float(np.abs(s[k] - so[k]).max()) for k in KEYS) <= 1e-5 * scale


@pytest.mark.parametrize("count,m", [(4096, 20), (2048, 100), (1024, 500), (64, 200), (300, 1500)])
def test_default_tiles_are_near_the_best_workgroup(count, m):
    """The workgroup that the batch chooses for itself, against the others:
    at most 1.25 times the fastest (one of 1024 threads for every batch took
    4.5 times the time of narrow ones with many small instances)."""
    insts = [_instance(m, 2 * m, min(1.0, 4.0 / m), 41 + i) for i in range(4)]
    for i in insts:  # no dense segments
        A = sp.random(i["m"], i["n"], density=min(1.0, 6.0 / m), random_state=i["m"], format="csr")
        i.update(row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data - 0.5)
    with Batch((insts * ((count + 3) // 4))[:count], precision="mixed", eps=0.0) as b:
        threads, lanes = b.get_tiles()
        own = min(b.time(-1, 50) for _ in range(3))
        others = {}
        for t in (64, 128, 256, 512, 1024):
            b.set_tiles(t, [2 if t < 256 else 4, 0, 1, 0, 1, 0, 1, 0])
            others[t] = min(b.time(-1, 50) for _ in range(3))
    sys.__stderr__.write(f"[gpu-test] batch {count} x {m}: own {threads} {lanes} {own:.3f} ms, {others}\n")
    assert own <= 1.25 * min(others.values()), (threads, own, others)

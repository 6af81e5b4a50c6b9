"""The launch-shape searches: slab counts of the single-problem solver."""
import pytest

from paper_2203_05027_amd import autotune
from paper_2203_05027_amd import instances as I

pytestmark = pytest.mark.gpu


def test_slab_search_picks_the_fastest_measured_count(tmp_path):
    inst = I.lp_instance(300_000, 600_000, 8, seed=51)
    cache = str(tmp_path / "tiles.json")
    rec = autotune.tune_slabs(inst, "fp64", iters=10, cache_path=cache)
    assert not rec["cached"]
    trials = rec["trials"]
    assert {t["slabs"] for t in trials} == {1, 2, 4, 8}
    assert rec["ms_row"] == min(t["ms_row"] for t in trials)
    assert rec["ms_col"] == min(t["ms_col"] for t in trials)
    again = autotune.tune_slabs(inst, "fp64", iters=10, cache_path=cache)
    assert again["cached"] and again["slabs_row"] == rec["slabs_row"] and again["slabs_col"] == rec["slabs_col"]


def test_the_shape_says_which_products_run():
    from paper_2203_05027_amd.solver import Solver, Standard
    for m, n, k, product in ((330_001, 640_009, 9, "binned"), (5000, 12_000, 80, "staged"), (3000, 6000, 5, "lanes")):
        inst = I.lp_instance(m, n, k, seed=54)
        with Solver.from_instance(inst, eps=0.0) as s:
            shape = s.launch_shape()
            assert shape["product_row"] == shape["product_col"] == product, shape
            assert shape["slabs_row"] == shape["slabs_col"] == 1
        if product == "binned":
            with Standard.from_instance(inst, cg_iters=1) as s:
                assert s.launch_shape() == {"slabs_row": 1, "slabs_col": 1}
            with Solver.from_instance(inst, eps=0.0, slabs_row=4, slabs_col=2) as s:
                shape = s.launch_shape()
                assert shape["product_row"] == shape["product_col"] == "slabs" and shape["slabs_row"] == 4


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_slab_search_times_the_automatic_choice(tmp_path, precision):
    """Where the solver's own choice is a product without slabs, the record
    does not take it away: a solver created with it is as fast as one without."""
    from paper_2203_05027_amd.solver import Solver
    inst = I.lp_instance(600_000, 1_000_000, 10, seed=52)
    rec = autotune.tune_slabs(inst, precision, iters=20, cache_path=str(tmp_path / "tiles.json"))
    ms = []
    for kw in ({}, dict(slabs_row=rec["slabs_row"], slabs_col=rec["slabs_col"])):
        with Solver.from_instance(inst, precision=precision, eps=0.0, **kw) as s:
            s.iterate(2)
            ms.append(min(sum(s.time_kernels(20)) for _ in range(3)))
            shape = s.launch_shape()
            if not kw:
                assert shape["product_row"] == shape["product_col"] == "binned"
                assert shape["slabs_row"] == shape["slabs_col"] == 1
    assert ms[1] <= 1.05 * ms[0], (rec, ms)


def test_slab_search_keeps_the_resident_path(tmp_path):
    rec = autotune.tune_slabs(I.lp_instance(500, 1000, 5, seed=53), "fp64", iters=5, cache_path=str(tmp_path / "t.json"))
    assert rec["slabs_row"] == 0 and rec["slabs_col"] == 0


def test_a_shape_for_one_pass_leaves_the_other_automatic():
    import oracle
    import numpy as np
    from paper_2203_05027_amd.solver import Solver
    inst = I.lp_instance(330_001, 640_009, 9, seed=54)
    o = oracle.Oracle.from_instance(inst)
    o.iterate(11)
    so = o.state()
    for kw, products in ((dict(slabs_row=4), ("slabs", "binned")), (dict(lanes_col=4, slabs_col=1), ("binned", "lanes")),
                         (dict(slab_kernel="lanes"), ("slabs", "slabs"))):
        with Solver.from_instance(inst, eps=0.0, check_every=5, **kw) as s:
            shape = s.launch_shape()
            assert (shape["product_row"], shape["product_col"]) == products, shape
            s.iterate(11)
            g, r = s.solution(), s.residuals()
        for k in g:
            assert np.abs(g[k] - so[k]).max() <= 1e-9 * max(np.abs(so[k]).max(), 1e-30), (kw, k)
        assert abs(r["r_prim"] - o.residuals()["r_prim"]) <= 1e-9

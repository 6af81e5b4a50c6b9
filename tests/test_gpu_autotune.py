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

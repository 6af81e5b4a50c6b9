"""The one-launch set-up of the call that allocates nothing, at the sizes where
it can go wrong (one row or column, empty rows and columns, more columns than
its scan takes at once, long columns, no entries), against the call that
prepares everything with the general kernels: bitwise the same outputs and
residuals, at every place the last iterate can have in the checks' period."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2203_05027_amd.solver import solve

pytestmark = pytest.mark.gpu
KEYS = ("x", "z", "delta", "lambda")


def _instance(m, n, density, seed):
    rng = np.random.default_rng(seed)
    A = sp.random(m, n, density=density, random_state=rng, data_rvs=rng.standard_normal, format="lil")
    if m > 3 and n > 3:
        A[m // 2] = 0.0
        A[:, n // 3] = 0.0
        A[0] = 0.0
        A[: min(m, 400), n - 1] = 0.1
    A = A.tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    return dict(m=m, n=n, row_ptr=A.indptr.astype(np.int64), col_idx=A.indices.astype(np.int32), val=A.data,
                b=A @ np.maximum(rng.standard_normal(n), 0.0), c=A.T @ rng.standard_normal(m) + rng.uniform(0, 1, n),
                n_orth=n, soc_sizes=np.zeros(0, np.int32))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(1, 1, 1.0), (1, 3000, 0.5), (2500, 1, 0.8), (40, 60, 0.0), (63, 65, 0.3),
                                   (700, 1024, 0.004), (500, 1025, 0.004), (1030, 2100, 0.0015), (150, 331, 0.03)])
def test_noalloc_setup_equals_the_general_one(shape, precision):
    inst = _instance(*shape, seed=shape[0] + shape[1])
    for iters, full in ((0, 0), (1, 0), (20, 0), (20, 1), (23, 0)):
        kw = dict(precision=precision, eps=0.0, check_every=10, full_checks=full)
        rc_a, a, ra = solve(inst, iters, **kw)
        rc_b, b, rb = solve(inst, iters, noalloc=True, **kw)
        assert rc_a == rc_b == 0
        for k in KEYS:
            assert np.array_equal(a[k], b[k]), (iters, k)
        assert ra == rb, iters


def test_a_query_after_a_skipped_check_decides_nothing():
    """An empty column with a cost of 1e200: the primal half of every check is
    finite and fails, the column half overflows, and only a check that is not
    skipped may stop the run for it."""
    inst = _instance(40, 90, 0.1, 3)
    c = inst["c"].copy()
    c[inst["n"] // 3] = 1e200
    inst = dict(inst, c=c)
    for iters in (10, 15, 20):
        rc_a, a, ra = solve(inst, iters, eps=0.0, check_every=10)
        rc_b, b, rb = solve(inst, iters, noalloc=True, eps=0.0, check_every=10)
        assert rc_a == rc_b
        for k in KEYS:
            assert np.array_equal(a[k], b[k], equal_nan=True), (iters, k)
        assert repr(ra) == repr(rb), iters

"""The family's blocks of 32 segments where they can go wrong: blocks whose
entries do not fit LDS, segments longer than a block holds, empty segments,
last blocks that are not full, groups of padding instances and groups that
have stopped."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from paper_2203_05027_amd.solver import Family

pytestmark = pytest.mark.gpu
KEYS = ("x", "z", "delta", "lambda")


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _family(m, n, k, seed, nb):
    rng = np.random.default_rng(seed)
    A = sp.random(m, n, density=k / m, random_state=rng, data_rvs=rng.standard_normal, format="lil")
    A[3, : n - 5] = 0.05          # a row longer than a block's LDS holds
    A[:, 11] = 0.03               # and a long column
    A[m // 2] = 0.0               # an empty row
    A[:, n - 1] = 0.0             # and an empty column
    A = A.tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    c = A.T @ rng.standard_normal(m) + rng.uniform(0.0, 1.0, n)
    b = np.stack([A @ np.maximum(rng.standard_normal(n), 0.0) for _ in range(nb)])
    return A, b, c


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m,n,k,B,nb", [(33, 65, 20, 64, 20), (700, 1603, 45, 192, 97), (2501, 4099, 6, 128, 128)])
def test_blocks_match_oracle(m, n, k, B, nb, precision):
    A, b, c = _family(m, n, k, 91 + m, nb)
    args = (m, n, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data, c)
    with Family(*args, B=B, precision=precision, eps=0.0, check_every=7) as F:
        F.set_rhs(b)
        F.iterate(30)
        sol, res = F.solution(), F.residuals()
    tol = 1e-9 if precision == "fp64" else 1e-5
    worst = 0.0
    for l in (0, 1, nb // 2, nb - 1):
        o = oracle.Oracle(m, n, args[2], args[3], args[4], b[l], c, n, np.zeros(0, np.int32))
        o.iterate(30)
        s = o.state()
        worst = max(worst, max(rel(sol[q][l], s[q]) for q in KEYS))
        assert res[l]["status"] == "running" and res[l]["iter"] == 30
    sys.__stderr__.write(f"[gpu-test] family blocks m={m} B={B} {precision}: {worst}\n")
    assert worst <= tol


def test_stopped_groups_are_left_alone():
    """Members of one group stop (max_iter after a refill is each member's
    own); the others go on, and the stopped ones keep their iterates."""
    m, n, nb = 700, 1603, 64
    A, b, c = _family(m, n, 6, 97, nb)
    args = (m, n, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data, c)
    with Family(*args, B=64, precision="mixed", eps=0.0, check_every=5, max_iter=20) as F:
        F.set_rhs(b)
        assert F.iterate(20) == 0
        F.refill(list(range(32, 64)), b[32:])
        before = F.solution()
        assert F.iterate(10) == 32
        after, res = F.solution(), F.residuals()
    for q in KEYS:
        assert np.array_equal(before[q][:32], after[q][:32]), q
        assert not np.array_equal(before[q][32:], after[q][32:]), q
    assert {r["status"] for r in res[:32]} == {"max_iter"} and {r["iter"] for r in res[32:]} == {10}

"""The FP32 matrix-core GEMM and the PCA fit at the sizes where they can go
wrong: edges of the 64 x 64 x 32 tiles, k split within workgroups and not,
every operand order, strides that are not one; odd, smallest and rank-deficient
eigenproblems."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


def _bound(A, B, K):
    """Any order of FP32 products and sums: (K + 2) u sum_k |a_ik| |b_kj|."""
    return (K + 2) * U32 * (A.abs().double() @ B.abs().double()) + 1e-30


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 65, 31), (64, 64, 32), (65, 130, 33), (200, 3, 4096),
                                   (17, 70, 2053), (513, 1025, 100)])
def test_gemm_tile_edges(M, N, K, tA, tB):
    import torch
    from paper_2203_05027_amd import learn
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7 + N * 3 + K)
    A = torch.randn(M, K, generator=g, device="cuda")
    B = torch.randn(K, N, generator=g, device="cuda")
    C0 = torch.randn(M, N, generator=g, device="cuda")
    As, Bs = (A.t().contiguous() if tA else A), (B.t().contiguous() if tB else B)
    C = C0.clone()
    learn.gemm(As, Bs, C, alpha=0.5, beta=-2.0, transA=tA, transB=tB)
    ref = 0.5 * (A.double() @ B.double()) - 2.0 * C0.double()
    err = (C.double() - ref).abs()
    assert bool((err <= _bound(A, B, K) + 4 * U32 * C0.abs().double()).all()), float(err.max())


def test_gemm_general_strides_and_unaligned_operands():
    import torch
    from paper_2203_05027_amd import learn
    from paper_2203_05027_amd.solver import lib
    M, N, K = 77, 90, 150
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    bufA = torch.randn(M * K * 2 + 1, generator=g, device="cuda")
    bufB = torch.randn(K * N * 3 + 3, generator=g, device="cuda")
    learn._bind()
    for a_off, a_rs, a_cs, b_off, b_rs, b_cs in [(0, 2 * K, 2, 0, 3 * N, 3), (1, K, 1, 3, N, 1), (1, 1, M, 1, 1, K),
                                                 (0, 2, 2 * M, 1, N + 1, 1)]:
        A = torch.as_strided(bufA, (M, K), (a_rs, a_cs), a_off)
        B = torch.as_strided(bufB, (K, N), (b_rs, b_cs), b_off)
        C = torch.full((M, N + 5), 7.0, device="cuda")  # ldc > N: the margin is left alone
        p = lambda t, o=0: ctypes.c_void_p(t.data_ptr() + 4 * o)
        rc = lib().gemm_f32(M, N, K, p(bufA, a_off), a_rs, a_cs, p(bufB, b_off), b_rs, b_cs, p(C), N + 5, 1.0, 0.0, None)
        assert rc == 0
        err = (C[:, :N].double() - A.double() @ B.double()).abs()
        assert bool((err <= _bound(A, B, K)).all()), float(err.max())
        assert bool((C[:, N:] == 7.0).all())


@pytest.mark.parametrize("N,D,k,over", [(37, 50, 20, 32), (2, 5, 1, 0), (1, 7, 1, 3), (70, 41, 41, 32), (300, 200, 8, 9)])
def test_pca_spans_and_odd_sizes(N, D, k, over):
    """Samples of rank k plus noise 1e-3 of its smallest direction: mean,
    singular values and the reconstruction of an FP64 decomposition (FP32
    data and products through five of them: 1e-4); rank-k inputs that fill
    the whole space come back whole."""
    import torch
    from paper_2203_05027_amd import learn
    rng = np.random.default_rng(N + D)
    r = min(k, N, D)
    Y = (rng.standard_normal((N, r)) @ rng.standard_normal((r, D)) + rng.standard_normal(D)).astype(np.float32)
    Y += (1e-3 * rng.standard_normal((N, D))).astype(np.float32)
    mean, basis, sv = learn.pca_fit(torch.from_numpy(Y).cuda(), k, oversample=over)
    m = Y.astype(np.float64).mean(0)
    Uo, so, Vo = np.linalg.svd(Y - m, full_matrices=False)
    assert np.abs(mean.cpu().numpy() - m).max() <= 1e-5 * max(np.abs(m).max(), 1.0)
    top = max(so[0], 1e-30)
    assert np.abs(sv[: min(k, so.size)] - so[:k]).max() <= 1e-4 * top + 1e-4
    B = basis.cpu().numpy().astype(np.float64)
    back = (Y - m) @ B.T @ B
    want = (Uo[:, :k] * so[:k]) @ Vo[:k]
    assert np.linalg.norm(back - want) <= 2e-3 * np.linalg.norm(want) + 1e-3


def _spectrum(N, D, s, seed):
    """Samples whose centered singular values are s (and a mean), in FP32; the values are made again in FP64."""
    rng = np.random.default_rng(seed)
    U = rng.standard_normal((N, s.size))
    U = np.linalg.qr(U - U.mean(0))[0]
    V = np.linalg.qr(rng.standard_normal((D, s.size)))[0]
    return ((U * s) @ V.T + rng.standard_normal(D)).astype(np.float32)


def _fit(Y, k, over):
    import torch
    from paper_2203_05027_amd import learn
    mean, basis, sv = learn.pca_fit(torch.from_numpy(Y).cuda(), k, oversample=over)
    return Y - mean.cpu().numpy().astype(np.float64), basis.cpu().numpy().astype(np.float64), sv


# FP32 samples and products: an absolute error of some tens of units of the
# largest singular value's rounding
SV_TOL = 64 * U32


@pytest.mark.parametrize("decades", [3.4, 4.2])
@pytest.mark.parametrize("N,D,k,over", [(300, 8, 8, 32), (60, 200, 8, 0), (100, 100, 4, 0), (500, 400, 48, 16)])
def test_pca_keeps_small_directions(N, D, k, over, decades):
    """Singular values over three and four decades: each of them, its
    direction and orthonormal rows."""
    s = np.logspace(0.0, -decades, k) * np.sqrt(N)
    Yc, B, sv = _fit(_spectrum(N, D, s, N + k), k, over)
    _, so, Vo = np.linalg.svd(Yc, full_matrices=False)
    assert np.abs(sv - so[:k]).max() <= SV_TOL * so[0]
    assert np.abs(B @ B.T - np.eye(k)).max() <= 1e-5
    cos = np.abs((B * Vo[:k]).sum(1))
    # mixing with its neighbours: the error over the gap to the next value
    gap = np.minimum(so[:k] - np.append(so[1:k], 0.0), np.append(np.inf, so[: k - 1] - so[1:k]))
    assert (cos >= 1.0 - (SV_TOL * so[0] / gap) ** 2 - 1e-5).all(), (cos, gap / so[0])


@pytest.mark.parametrize("N,D,rank,noise,k,over", [(300, 200, 10, 0.0, 32, 32), (300, 200, 32, 0.0, 64, 32),
                                                   (300, 200, 10, 1e-3, 32, 32), (40, 50, 10, 0.0, 32, 32),
                                                   (20, 30, 0, 0.0, 4, 3), (1, 7, 0, 0.0, 1, 3), (2, 5, 1, 0.0, 2, 3),
                                                   (64, 64, 63, 0.0, 64, 0)])
def test_pca_beyond_the_rank(N, D, rank, noise, k, over):
    """More components than the samples have directions: orthonormal rows all
    the same, the samples come back from them, and zeros as singular values."""
    rng = np.random.default_rng(N + D + rank)
    Y = (rng.standard_normal((N, rank)) @ rng.standard_normal((rank, D)) if rank else np.zeros((N, D)))
    Y = (Y + noise * rng.standard_normal((N, D)) + rng.standard_normal(D)).astype(np.float32)
    Yc, B, sv = _fit(Y, k, over)
    _, so, Vo = np.linalg.svd(Yc, full_matrices=False)
    top = max(so[0], 1e-30)
    assert np.abs(B @ B.T - np.eye(k)).max() <= 1e-5
    want = np.zeros(k)
    want[: min(k, so.size)] = so[:k]
    assert np.abs(sv - want).max() <= SV_TOL * top + 1e-5 * np.abs(Y).max()
    best = np.sqrt((so[k:] ** 2).sum())  # what no k directions can hold
    assert np.linalg.norm(Yc - Yc @ B.T @ B) <= 1.05 * best + 1e-5 * np.linalg.norm(Yc) + 1e-5 * np.abs(Y).max()


@pytest.mark.parametrize("scale", [1e-15, 1e15])
def test_pca_of_very_small_and_large_samples(scale):
    """Squares that leave FP32's range."""
    Y = _spectrum(90, 60, np.logspace(0.0, -2.0, 6) * 9.0, 8)
    Yc, B, sv = _fit((Y * np.float32(scale)).astype(np.float32), 6, 8)
    so = np.linalg.svd(Yc, compute_uv=False)
    assert np.abs(sv - so[:6]).max() <= SV_TOL * so[0]
    assert np.abs(B @ B.T - np.eye(6)).max() <= 1e-5


def test_pca_of_samples_with_nan_says_so():
    Y = _spectrum(90, 60, np.ones(6), 9)
    Y[3, 5] = np.nan
    _, B, sv = _fit(Y, 6, 8)
    assert np.isnan(sv).all() and np.isnan(B).all()

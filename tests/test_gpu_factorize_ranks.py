"""xkv_factorize_svd at ranks on both sides of its block sizes: the Cholesky panels (32 columns, with and without bounds checks), their
row tiles of 16 and the column blocks of 16 of the eigen-solver; several sequences, rank-deficient input.

Checked on what holds for every spectrum, converged or not: B B^T = I, A = X B^T, A^T A diagonal and descending with the
returned sigma^2 on its diagonal.  Bounds (fp32 storage): the orthonormalisation ends at fp32 rounding of unit vectors
(1e-5 as in the other factorization tests); the Rayleigh-Ritz matrix is formed from fp32 products, which leaves
1e-6 .. 1e-5 of the largest eigenvalue beside the diagonal (1e-4 used).  The full-rank inputs are conditioned for that: the
singular values fall off as i^-0.6 along orthonormal directions, so those of C = X^T X span at most 1024^1.2 = 4e3 and
C V keeps every direction far above fp32 rounding (4e3 * 2^-24 = 2.4e-4 of its length).  With random instead of orthonormal
directions and r = n = 1024 C is singular to fp32 (its spread was above 1e9) and the orthonormality of the last rows is
a matter of chance: 1e-5 to 5e-2 over five seeds, with one-panel substitution as well as with the inverted panel."""
import numpy as np
import pytest

from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


def factorize(X, G, H_kv, d_h, L, r, iters):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    batch, n = len(X), G * H_kv * d_h
    shape = xb.Shape(G=G, H_kv=H_kv, H_q=H_kv, d_h=d_h, r_k=r, r_v=r, L=L, k=1, batch=batch, dtype="f32")
    Xd = torch.from_numpy(X).cuda()
    A = torch.zeros((batch, L, r), device="cuda")
    B = torch.zeros((batch, G, r, H_kv * d_h), device="cuda")
    sigma = torch.zeros((batch, r), device="cuda")
    ws = torch.full((xb.xkv_factorize_workspace_bytes(shape, r),), 255, dtype=torch.uint8, device="cuda")
    xb.xkv_factorize_svd(shape, Xd, r, r, iters, 11, A, B, sigma, ws)
    torch.cuda.synchronize()
    return (A.double().cpu().numpy(), B.double().cpu().numpy().transpose(0, 2, 1, 3).reshape(batch, r, n),
            sigma.double().cpu().numpy())


@pytest.mark.parametrize("r,batch,rank", [
    (2, 1, None), (15, 1, None), (16, 3, None), (17, 1, None), (31, 1, None), (32, 1, None), (33, 2, None), (47, 1, None),
    (48, 1, None), (65, 1, None), (129, 1, None), (40, 1, 12), (100, 2, 33),
    (496, 1, None), (511, 1, None), (512, 1, None), (513, 1, None), (527, 1, None), (545, 1, None), (1024, 1, None),
])
def test_ranks_around_the_block_sizes(r, batch, rank):
    G, H_kv, d_h = (2, 4, 128) if r > 128 else (1, 3, 64)
    L, n = (1100 if r > 128 else 300), G * H_kv * d_h
    rng = np.random.default_rng(1000 + r)
    m = min(L, n) if rank is None else rank
    directions = np.linalg.qr(rng.standard_normal((n, n)))[0]
    X = np.zeros((batch, G, H_kv, L, d_h), np.float32)
    for b in range(batch):
        flat = (rng.standard_normal((L, m)) * (1.0 + np.arange(m)) ** -0.6) @ directions[:m]
        X[b] = flat.reshape(L, G, H_kv, d_h).transpose(1, 2, 0, 3)
    A, B, sigma = factorize(X, G, H_kv, d_h, L, r, 3)
    assert np.isfinite(A).all() and np.isfinite(B).all() and np.isfinite(sigma).all()
    for b in range(batch):
        flat = X[b].astype(np.float64).transpose(2, 0, 1, 3).reshape(L, n)
        if rank is None:
            assert np.abs(B[b] @ B[b].T - np.eye(r)).max() <= 1e-5
        ref_A = flat @ B[b].T
        assert np.abs(A[b] - ref_A).max() <= 1e-5 * np.abs(ref_A).max()
        gram = A[b].T @ A[b]
        lam = np.diag(gram)
        assert np.abs(gram - np.diag(lam)).max() <= 1e-4 * lam.max()
        assert (sigma[b][1:] <= sigma[b][:-1]).all()
        np.testing.assert_allclose(sigma[b] ** 2, lam, rtol=0, atol=1e-4 * lam.max())


def test_a_nan_in_the_input_stays_a_value():
    """The directions are ordered by their singular values; without an order among NaN the places of the list stayed
    unwritten and were used as row numbers all the same.  The other sequence of the batch is not touched."""
    G, H_kv, d_h, L, r = 1, 2, 64, 300, 40
    n = G * H_kv * d_h
    rng = np.random.default_rng(3)
    X = rng.standard_normal((2, G, H_kv, L, d_h)).astype(np.float32)
    X[0, 0, 1, 17, 5] = np.nan
    A, B, sigma = factorize(X, G, H_kv, d_h, L, r, 3)
    assert np.isnan(sigma[0]).any()
    assert np.isfinite(A[1]).all() and np.isfinite(B[1]).all()
    assert np.abs(B[1] @ B[1].T - np.eye(r)).max() <= 1e-5
    flat = X[1].astype(np.float64).transpose(2, 0, 1, 3).reshape(L, n)
    ref_A = flat @ B[1].T
    assert np.abs(A[1] - ref_A).max() <= 1e-5 * np.abs(ref_A).max()


@pytest.mark.parametrize("r,batch", [(64, 3), (96, 1), (128, 1), (130, 1), (160, 2), (256, 1)])
def test_ranks_of_whole_pairs_of_blocks(r, batch):
    """The eigen-solver leaves its bounds checks out where r is a multiple of 32; 128 positions of J^T per workgroup."""
    test_ranks_around_the_block_sizes(r, batch, None)

"""The merge of split partials, through full attention in fp32: from one partial to several rounds of its loads, up to 64
partials, up to 256 and more, columns in fours and one at a time in groups of 8 to 256 threads, and the partials of an
uncompressed tail as a second set.  Against fp64 NumPy."""
import numpy as np
import pytest

from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


# the general kernel leaves four partials per 256 tokens here: 4 of them at L = 1 and 40, 12 at 700, 64 at 4096, 68 at 4100, 144 at
# 9000, 256 at 16384, 268 at 17000 and 508 at 32257
SHAPES = [(d_h, 2, 2, L) for d_h in (6, 30, 64, 65, 70, 100, 128, 130, 255, 256) for L in (1, 40, 700, 9000)] + \
         [(d_h, 1, 1, L) for d_h in (6, 70, 255, 256) for L in (4096, 4100, 16384, 17000, 32257)]


@pytest.mark.parametrize("d_h,H_kv,batch,L", SHAPES)
def test_dense_over_many_splits(d_h, H_kv, batch, L):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    H_q = 2 * H_kv
    rng = np.random.default_rng(d_h * 10 + L)
    K, V = (rng.standard_normal((batch, H_kv, L, d_h)).astype(np.float32) for _ in range(2))
    q = rng.standard_normal((batch, H_q, d_h)).astype(np.float32)
    shape = xb.Shape(G=1, H_kv=H_kv, H_q=H_q, d_h=d_h, r_k=4, r_v=4, L=L, k=1, batch=batch, dtype="f32")
    dev = [torch.from_numpy(x).cuda() for x in (K, V, q)]
    out = torch.zeros((batch, H_q, d_h), device="cuda")
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    xb.xkv_dense_decode(shape, dev[0], dev[1], dev[2], out, ws)
    torch.cuda.synchronize()
    z = np.einsum("bgtj,bgrj->bgrt", K.astype(np.float64), q.astype(np.float64).reshape(batch, H_kv, H_q // H_kv, d_h)) / np.sqrt(d_h)
    p = np.exp(z - z.max(-1, keepdims=True))
    want = np.einsum("bgrt,bgtj->bgrj", p / p.sum(-1, keepdims=True), V.astype(np.float64)).reshape(batch, H_q, d_h)
    # logits to d_h 2^-24 |z| and the weighted mean of values of size about 4: well below 1e-5 of the largest
    np.testing.assert_allclose(out.double().cpu().numpy(), want, rtol=0, atol=2e-5 * np.abs(V).max())


@pytest.mark.parametrize("d_h,r", [(64, 32), (64, 21), (100, 9), (256, 5)])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 33, 64, 65, 200])
def test_general_gather_over_its_splits(d_h, r, k):
    """The general gather kernel splits a list down to 16 rows per workgroup where the partials have room: every remainder of
    a round, and ranks that its unrolled loops do not divide."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    G, H_kv, H_q, L, batch, layer = 2, 2, 4, 1500, 2, 1
    rng = np.random.default_rng(d_h * 1000 + k)
    A_k, A_v = (rng.standard_normal((batch, L, r)).astype(np.float32) for _ in range(2))
    B_k, B_v = ((rng.standard_normal((batch, G, r, H_kv * d_h)) / np.sqrt(r)).astype(np.float32) for _ in range(2))
    q = rng.standard_normal((batch, H_q, d_h)).astype(np.float32)
    idx = np.stack([[np.sort(rng.permutation(L)[:k]) for _ in range(H_kv)] for _ in range(batch)]).astype(np.int32)
    shape = xb.Shape(G=G, H_kv=H_kv, H_q=H_q, d_h=d_h, r_k=r, r_v=r, L=L, k=k, batch=batch, dtype="f32")
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (A_k, A_v, B_k, B_v, q, idx)]
    out = torch.zeros((batch, H_q, d_h), device="cuda")
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    xb.xkv_gather_attend(shape, layer, *dev, out, ws)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    for b in range(batch):
        for h in range(H_q):
            g = h // (H_q // H_kv)
            cols, rows = slice(g * d_h, (g + 1) * d_h), idx[b, g]
            K = A_k[b, rows].astype(np.float64) @ B_k[b, layer][:, cols]
            V = A_v[b, rows].astype(np.float64) @ B_v[b, layer][:, cols]
            z = K @ q[b, h].astype(np.float64) / np.sqrt(d_h)
            p = np.exp(z - z.max())
            # rows of K and V to r 2^-24 of the sums of absolute products, logits to d_h 2^-24 of theirs: 1e-5 of the largest
            np.testing.assert_allclose(got[b, h], (p / p.sum()) @ V, rtol=0, atol=5e-5 * np.abs(V).max())


@pytest.mark.parametrize("d_h,L,k,T", [(64, 1500, 200, 300), (70, 1500, 200, 300), (130, 40000, 3000, 1100), (256, 40000, 3000, 1100)])
def test_selected_rows_and_tail_in_one_merge(d_h, L, k, T):
    """Partials of the selected rows and of the tail together, fewer and more than 64 of them."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    H_kv, H_q, r = 1, 2, 8
    rng = np.random.default_rng(d_h + L)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    A_k, A_v, B_k, B_v, q = f32(1, L, r), f32(1, L, r), f32(1, 1, r, d_h), f32(1, 1, r, d_h), f32(1, H_q, d_h)
    K_t, V_t = f32(1, 1, T, d_h), f32(1, 1, T, d_h)
    shape = xb.Shape(G=1, H_kv=H_kv, H_q=H_q, d_h=d_h, r_k=r, r_v=r, L=L, k=k, batch=1, dtype="f32")
    dev = [torch.from_numpy(x).cuda() for x in (A_k, A_v, B_k, B_v, q, K_t, V_t)]
    out, idx = torch.zeros((1, H_q, d_h), device="cuda"), torch.zeros((1, 1, k), dtype=torch.int32, device="cuda")
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    xb.xkv_sr_decode_tail(shape, 0, *dev, T, out, idx, None, ws)
    torch.cuda.synchronize()
    rows = idx.cpu().numpy()[0, 0]
    K = np.concatenate([A_k[0, rows].astype(np.float64) @ B_k[0, 0], K_t[0, 0]])
    V = np.concatenate([A_v[0, rows].astype(np.float64) @ B_v[0, 0], V_t[0, 0]])
    for h in range(H_q):
        z = K @ q[0, h].astype(np.float64) / np.sqrt(d_h)
        p = np.exp(z - z.max())
        # as above; logits of the reconstructed rows are r times larger
        np.testing.assert_allclose(out.double().cpu().numpy()[0, h], (p / p.sum()) @ V, rtol=0, atol=5e-5 * np.abs(V).max())

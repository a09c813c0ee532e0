"""The general score kernel over its head blocks (4 where a KV head has no more query heads, else 8) and ranks that its
unrolled loop does not divide, against fp64: p = B q (d_h terms) and s = A p (r terms), each sum rounded at most once per
term in fp32, so |error| <= (d_h + r + 2) 2^-24 scale |A| (|B| |q|) up to second order (3x used)."""
import numpy as np
import pytest

from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rep", [1, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("r", [1, 7, 8, 33])
def test_scores_against_fp64(n_rep, r):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    G, H_kv, d_h, L, batch, layer = 2, 2, 40, 259, 2, 1
    H_q = H_kv * n_rep
    rng = np.random.default_rng(n_rep * 100 + r)
    A = rng.standard_normal((batch, L, r)).astype(np.float32)
    B = rng.standard_normal((batch, G, r, H_kv * d_h)).astype(np.float32)
    q = rng.standard_normal((batch, H_q, d_h)).astype(np.float32)
    shape = xb.Shape(G=G, H_kv=H_kv, H_q=H_q, d_h=d_h, r_k=r, r_v=r, L=L, k=1, batch=batch, dtype="f32")
    dev = [torch.from_numpy(x).cuda() for x in (A, B, q)]
    S = torch.zeros((batch, H_kv, L), device="cuda")
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    xb.xkv_score(shape, layer, *dev, S, ws)
    torch.cuda.synchronize()
    got, scale = S.double().cpu().numpy(), 1.0 / np.sqrt(d_h)
    for b in range(batch):
        for g in range(H_kv):
            Bg = B[b, layer][:, g * d_h:(g + 1) * d_h].astype(np.float64)
            qs = q[b, g * n_rep:(g + 1) * n_rep].astype(np.float64).T
            s = scale * (A[b].astype(np.float64) @ (Bg @ qs))
            size = scale * (np.abs(A[b]).astype(np.float64) @ (np.abs(Bg) @ np.abs(qs)))
            assert (np.abs(got[b, g] - s.max(1)) <= 3 * (d_h + r + 2) * 2.0 ** -24 * size.max(1)).all()

"""The score kernel for ranks above 256 over up to 1024 token tiles: ragged last tiles and wavefronts without one, every number of
rank steps, every number of heads per KV head, and both sides of the line to the long-stream kernel, there with four and eight
wavefronts."""
import numpy as np
import pytest

import oracle
from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r_k,H_kv,n_rep,L,batch", [
    (272, 2, 1, 5, 1), (272, 3, 16, 33, 1), (288, 5, 2, 129, 2), (512, 8, 4, 1025, 3), (512, 2, 3, 4096, 1), (640, 4, 8, 97, 1), (768, 4, 5, 700, 1),
    (768, 3, 6, 31, 1), (384, 2, 7, 1000, 1), (512, 2, 4, 32768, 1), (512, 2, 4, 32769, 1), (144, 2, 4, 33000, 1),
    (192, 8, 4, 36000, 1), (512, 2, 4, 41005, 1), (768, 3, 4, 33900, 1)])
def test_score_ring(r_k, H_kv, n_rep, L, batch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = synth.Workload("score_ring", G=2, H_kv=H_kv, H_q=H_kv * n_rep, d_h=256, r_k=r_k, r_v=32, L=L, k=1, batch=batch, dtype="bf16",
                       a_scale=r_k ** -0.5, sigma_decay=0.8, q_scale=0.05)
    case = synth.make_case(w, seed=L + r_k)
    dev = synth.to_device(case, "bf16")
    shape = xb.Shape.of(w)
    ws = torch.empty(xb.xkv_absorbed_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    q = dev["q"][1].contiguous()
    S, S_fused = torch.empty((batch, H_kv, L), device="cuda"), torch.empty((batch, H_kv, L), device="cuda")
    S_heads = torch.empty((batch, H_kv, L), device="cuda")
    heads = torch.full((batch, H_kv, L, xb.head_pitch(shape)), 7.0, device="cuda")
    xb.xkv_score(shape, 1, dev["A_k"], dev["B_k"], q, S, ws)
    xb.xkv_head_scores(shape, 1, dev["A_k"], dev["B_k"], q, S_heads, heads, ws)
    out, idx = torch.empty((batch, w.H_q, w.d_h), device="cuda"), torch.empty((batch, H_kv, 1), dtype=torch.int32, device="cuda")
    xb.xkv_sr_decode(shape, 1, dev["A_k"], dev["A_v"], dev["B_k"], dev["B_v"], q, out, idx, S_fused, ws)
    assert torch.equal(S, S_fused) and torch.equal(S, S_heads)
    assert torch.equal(heads[..., :n_rep].amax(-1), S) and not heads[..., n_rep:].any()
    for b in range(batch):
        ref = oracle.pooled_scores(case["A_k"][b], case["B_k"][b, 1], case["q"][1, b], H_kv, oracle.default_scale(w.d_h))
        # P is held as two bf16 parts (2^-16 of it is lost, summed like sqrt(r_k) of them) and summed over at most 768 ranks in single
        # precision: far below 1e-4 of the largest score
        assert np.abs(S[b].cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max(), b

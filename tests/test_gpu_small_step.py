"""The one-launch step of small single-precision problems at the edges of its loops and of its range, against double precision, and
against the chained stages bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H_kv,n_rep,d_h,r_k,r_v,L,k,T,batch,shift", [
    (1, 4, 64, 32, 32, 512, 32, 0, 1, 0), (1, 1, 1, 1, 1, 1, 1, 0, 1, 0), (2, 5, 100, 33, 47, 63, 63, 1, 2, 0), (1, 16, 96, 64, 96, 1023, 100, 64, 1, 0),
    (2, 3, 256, 48, 32, 1025, 1, 0, 1, 0), (1, 4, 64, 48, 32, 4096, 1024, 10, 1, 0), (1, 4, 64, 64, 64, 4096, 300, 0, 1, 0),
    (8, 2, 128, 32, 1024, 200, 50, 0, 1, 0), (3, 7, 65, 40, 24, 900, 450, 33, 2, 1), (1, 4, 64, 63, 63, 4097, 64, 0, 1, 0)])
def test_small_step(H_kv, n_rep, d_h, r_k, r_v, L, k, T, batch, shift):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = synth.Workload("small_step", G=2, H_kv=H_kv, H_q=H_kv * n_rep, d_h=d_h, r_k=r_k, r_v=r_v, L=L, k=k, batch=batch, dtype="f32",
                       a_scale=1.0, sigma_decay=0.3, q_scale=0.3)
    case = synth.make_case(w, seed=L + k)
    dev = synth.to_device(case, "f32")
    rng = np.random.default_rng(L)
    tail = [rng.standard_normal((batch, H_kv, T, d_h)).astype(np.float32) for _ in "kv"]
    dt = [torch.from_numpy(x).cuda() if T else None for x in tail]
    A_k = dev["A_k"]
    if shift:  # rows off the 16-byte boundary
        buf = torch.empty(A_k.numel() + 4, device="cuda")
        buf[shift:shift + A_k.numel()] = A_k.reshape(-1)
        A_k = buf[shift:shift + A_k.numel()].view(A_k.shape)
    shape = xb.Shape.of(w)
    ws = xb.alloc_workspace(shape)
    q = dev["q"][1].contiguous()
    out, staged = torch.empty((batch, w.H_q, d_h), device="cuda"), torch.empty((batch, w.H_q, d_h), device="cuda")
    idx = torch.full((batch, H_kv, k), -1, dtype=torch.int32, device="cuda")
    S, S2 = torch.empty((batch, H_kv, L), device="cuda"), torch.empty((batch, H_kv, L), device="cuda")
    xb.xkv_sr_decode_tail(shape, 1, A_k, dev["A_v"], dev["B_k"], dev["B_v"], q, dt[0], dt[1], T, out, idx, S, ws)
    xb.xkv_score(shape, 1, A_k, dev["B_k"], q, S2, ws)
    assert torch.equal(S, S2)
    ids, got = idx.cpu().numpy(), out.cpu().numpy().astype(np.float64)
    for b in range(batch):
        for g in range(H_kv):
            np.testing.assert_array_equal(ids[b, g], oracle.select(S[b, g].cpu().numpy(), k))
        args = (case["A_k"][b], case["A_v"][b], case["B_k"][b, 1], case["B_v"][b, 1], case["q"][1, b], ids[b])
        ref = oracle.gather_attend_tail(*args, tail[0][b], tail[1][b]) if T else oracle.gather_attend(*args)
        # single-precision weights and sums of at most a few thousand terms
        assert np.abs(got[b] - ref).max() <= 2e-6 * max(np.abs(ref).max(), 1e-6), b
    if T == 0:
        xb.xkv_gather_attend(shape, 1, A_k, dev["A_v"], dev["B_k"], dev["B_v"], q, idx, staged, ws)
        assert torch.equal(out, staged)

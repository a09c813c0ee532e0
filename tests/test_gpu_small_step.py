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
    (8, 2, 128, 32, 1024, 200, 50, 0, 1, 0), (3, 7, 65, 40, 24, 900, 450, 33, 2, 1), (1, 4, 64, 63, 63, 4097, 64, 0, 1, 0),
    # scores and selection launched before it (from 163840 numbers of A^K on, up to two KV heads), and beside that line
    (1, 1, 64, 64, 40, 2050, 77, 5, 1, 0), (4, 3, 64, 64, 64, 2600, 100, 0, 2, 0), (1, 1, 64, 64, 40, 2600, 77, 5, 1, 0),
    (2, 3, 64, 64, 64, 2700, 100, 0, 2, 0), (2, 1, 64, 64, 40, 2560, 77, 5, 1, 0),
    # more pairs than compute units: four wavefronts each for given rows, more parts of a sum than threads; sixteen for more work
    (8, 2, 32, 16, 16, 64, 16, 0, 40, 0), (3, 5, 64, 24, 7, 100, 33, 0, 90, 0), (8, 4, 64, 32, 48, 90, 30, 3, 70, 0), (8, 4, 128, 96, 64, 70, 40, 0, 33, 0)])
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


@pytest.mark.parametrize("L,H_kv", [(512, 1), (4096, 1)])   # one launch; scores and selection on their own
def test_kernel_timing_does_not_change_the_step(L, H_kv):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = synth.Workload("small_step", G=1, H_kv=H_kv, H_q=4, d_h=64, r_k=48, r_v=32, L=L, k=40, batch=1, dtype="f32", a_scale=1.0,
                       sigma_decay=0.3, q_scale=0.3)
    dev = synth.to_device(synth.make_case(w, seed=L), "f32")
    shape, q = xb.Shape.of(w), dev["q"][0].contiguous()
    ws = xb.alloc_workspace(shape)
    idx = torch.empty((1, H_kv, w.k), dtype=torch.int32, device="cuda")

    def outputs():
        step, rows = torch.empty_like(q), torch.empty_like(q)
        xb.xkv_sr_decode(shape, 0, dev["A_k"], dev["A_v"], dev["B_k"], dev["B_v"], q, step, idx, None, ws)
        xb.xkv_gather_attend(shape, 0, dev["A_k"], dev["A_v"], dev["B_k"], dev["B_v"], q, idx, rows, ws)
        return step, rows

    plain = outputs()
    for stage in (xb.STAGE_SCORE, xb.STAGE_GATHER_ATTEND):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in ev:
            e.record()
        torch.cuda.synchronize()
        assert 0.0 <= ev[0].elapsed_time(ev[1])
        xb.xkv_profile_kernel(stage, ev[0].cuda_event, ev[1].cuda_event)
        try:
            timed = outputs()
        finally:
            xb.xkv_profile_kernel(stage, None, None)
        torch.cuda.synchronize()
        assert ev[0].elapsed_time(ev[1]) > 0.0
        assert all(torch.equal(a, b) for a, b in zip(plain, timed)), stage

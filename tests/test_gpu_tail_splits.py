"""The uncompressed tail inside the projection's launch: lengths at the edges of its splits, and tails that the matrix-core kernel
does not take (a launch of their own behind the selected rows)."""
import numpy as np
import pytest

import oracle
from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("T,batch", [(1, 2), (128, 2), (129, 2), (333, 2), (2048, 2), (2049, 2), (5000, 2), (700, 12), (513, 40)])  # (fewer splits each)
def test_tail_of_a_step(T, batch, shift):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = synth.LLAMA_GROUP.with_(L=700, k=90, r_k=64, r_v=96, batch=batch, G=1)
    case = synth.make_case(w, seed=T)
    dev = synth.to_device(case, "bf16")
    rng = np.random.default_rng(T)
    n = w.batch * w.H_kv * T * w.d_h
    tails, device = [], []
    for scale in (0.3, 1.0):
        x = synth.to_storage(rng.standard_normal((w.batch, w.H_kv, T, w.d_h)) * scale, "bf16")
        buf = torch.zeros(n + 8, dtype=torch.bfloat16, device="cuda")     # shift: off the 16-byte boundary
        buf[shift:shift + n] = synth.to_device({"x": x}, "bf16")["x"].reshape(-1)
        tails.append(x)
        device.append(buf[shift:shift + n].view(w.batch, w.H_kv, T, w.d_h))
    shape = xb.Shape.of(w)
    ws = xb.alloc_workspace(shape)
    out = torch.empty((w.batch, w.H_q, w.d_h), dtype=torch.bfloat16, device="cuda")
    idx = torch.empty((w.batch, w.H_kv, w.k), dtype=torch.int32, device="cuda")
    q = dev["q"][0].contiguous()
    xb.xkv_sr_decode_tail(shape, 0, dev["A_k"], dev["A_v"], dev["B_k"], dev["B_v"], q, device[0], device[1], T, out, idx, None, ws)
    torch.cuda.synchronize()
    got, ids = synth.storage_to_f64(synth.to_host(out)), idx.cpu().numpy()
    for b in range(w.batch):
        ref = oracle.gather_attend_tail(case["A_k"][b], case["A_v"][b], case["B_k"][b, 0], case["B_v"][b, 0], case["q"][0, b],
                                        ids[b], tails[0][b], tails[1][b])
        # bf16 weights, values and output: 2^-8 each at most, as for the step without a tail
        assert np.abs(got[b] - ref).max() <= 1e-2 * np.abs(ref).max()

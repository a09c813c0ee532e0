"""The selected-row kernel that keeps B_l out of its main loop (rows that are not rotated): stage call against the
definition -- reconstruct the selected rows, attend over them -- in double precision, where the kernel's tiles, rank groups
and merges have their edges.

Bound, element by element.  The kernel rounds two things to bf16, whose 8 significant bits make a rounding error of at most
2^-8 of the value: the weights w (the denominator is the sum of the unrounded ones) and the result.  So
|got - ref| <= 2^-8 (|ref| + sum_j w_j |v_j| / sum_j w_j).  The projected queries and the sums over rows are split into two
bf16 numbers (2^-17) and accumulated in single precision: 5 % on top, and 1e-6 of the largest value, cover these.
"""
import numpy as np
import pytest

import oracle
from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


def torch_mod():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def reference(A_k, A_v, B_k, B_v, q, rows, scale):
    """out, and sum_j w_j |v_j| / sum_j w_j, both [H_q][d_h]."""
    H_q, d_h = q.shape
    n_rep = H_q // len(rows)
    out, mag = np.zeros((H_q, d_h)), np.zeros((H_q, d_h))
    for g, r in enumerate(rows):
        if len(r) == 0:
            continue
        cols = slice(g * d_h, (g + 1) * d_h)
        K, V = A_k[r] @ B_k[:, cols], A_v[r] @ B_v[:, cols]
        for h in range(g * n_rep, (g + 1) * n_rep):
            z = scale * (K @ q[h])
            w = np.exp(z - z.max())
            out[h], mag[h] = w @ V / w.sum(), w @ np.abs(V) / w.sum()
    return out, mag


# (H_kv, n_rep, r_k, r_v, batch, k), then workgroups per compute unit and tiles of 128 rows per workgroup that the case is
# for: tests/test_plan.py checks on the host that it gets them (0 workgroups: the other kernel)
CASES = [
    # one row; both sides of a wavefront's 32 and of a tile's 128 rows; one rank group
    (1, 1, 16, 128, 1, 1, 1, 1), (2, 4, 128, 128, 1, 31, 1, 1), (1, 7, 256, 256, 2, 33, 1, 1), (2, 16, 256, 144, 1, 127, 1, 1),
    (3, 5, 144, 256, 1, 129, 1, 1),
    # three, four, five and six groups of A^V, unequal ranks, ragged last groups
    (2, 7, 384, 384, 1, 300, 1, 1), (1, 4, 512, 512, 1, 257, 1, 1), (1, 8, 384, 576, 1, 200, 1, 1), (2, 3, 640, 768, 1, 161, 1, 1),
    (1, 9, 528, 400, 1, 130, 1, 1),
    # two workgroups per compute unit (more than 256 tiles), the last tile ragged
    (8, 4, 512, 512, 5, 1000, 2, 1), (4, 7, 384, 384, 9, 1111, 2, 1), (8, 2, 128, 64, 6, 901, 2, 1), (8, 16, 256, 512, 5, 915, 2, 1),
    # several tiles per workgroup: the sums rescaled, requests from one tile's A^V to the next tile's A^K, and with more than
    # four tiles ids beyond the first 128 of a wavefront.  Two workgroups per compute unit, then one (r_k in rings of two and
    # of four groups, six groups of A^V)
    (8, 1, 16, 144, 128, 700, 2, 6), (8, 4, 512, 512, 16, 2200, 2, 3), (8, 2, 384, 384, 16, 1300, 2, 2),
    (8, 1, 640, 512, 32, 1100, 1, 9), (4, 2, 896, 512, 64, 300, 1, 3), (2, 16, 1024, 416, 128, 260, 1, 3), (8, 3, 512, 768, 32, 600, 1, 5),
    # more ranks of A^V than a wavefront keeps sums for: the rotated rows' kernel
    (1, 4, 128, 800, 1, 200, 0, 0),
]


@pytest.mark.parametrize("bits", [0, 4, 3])
@pytest.mark.parametrize("H_kv,n_rep,r_k,r_v,batch,k", [c[:6] for c in CASES])
def test_selected_rows_against_the_definition(H_kv, n_rep, r_k, r_v, batch, k, bits):
    torch = torch_mod()
    if bits and (r_k % 32 or r_v % 32):
        pytest.skip("quantised rows come in groups of 32 ranks")
    L = max(k + 5, 700)
    seqs = range(batch) if batch <= 9 else (0, batch // 2, batch - 1)  # that are compared
    w = synth.LLAMA_GROUP.with_(G=2, H_kv=H_kv, H_q=H_kv * n_rep, r_k=r_k, r_v=r_v, L=L, k=k, batch=batch, q_scale=3.0,
                                a_scale=1.0, sigma_decay=0.0)
    rng = np.random.default_rng(1000 * r_k + 10 * r_v + k + bits)
    d = w.d
    case = {"A_k": synth.to_storage(rng.standard_normal((batch, L, r_k)), "bf16"),
            "A_v": synth.to_storage(rng.standard_normal((batch, L, r_v)), "bf16"),
            "B_k": synth.to_storage(rng.standard_normal((batch, 2, r_k, d)) / np.sqrt(r_k), "bf16"),
            "B_v": synth.to_storage(rng.standard_normal((batch, 2, r_v, d)) / np.sqrt(r_v), "bf16"),
            "q": synth.to_storage(rng.standard_normal((2, batch, w.H_q, 128)), "bf16")}
    dev = synth.to_device(case, "bf16")
    idx = np.stack([np.stack([rng.choice(L, size=k, replace=False) for _ in range(H_kv)]) for _ in range(batch)]).astype(np.int32)
    idx[:, :, -1] = L - 1
    idx[:, :, k // 2] = idx[:, :, 0]          # ids need not be distinct
    counts = rng.integers(0, k + 1, size=(batch, H_kv)).astype(np.int32)
    counts[0, 0] = 0                          # a head without rows
    counts[-1, -1] = max(k - 1, 1)            # ... and one that ends in the last tile
    shape, layer = xb.Shape.of(w), 1
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    q = dev["q"][layer].contiguous()
    out = torch.empty((batch, w.H_q, 128), dtype=torch.bfloat16, device="cuda")
    A = {n: dev[n] for n in ("A_k", "A_v")}
    hat = {n: {b: synth.storage_to_f64(case[n][b]) for b in seqs} for n in ("A_k", "A_v")}
    if bits:
        for n, r in (("A_k", r_k), ("A_v", r_v)):
            A[n] = torch.empty((batch * L, xb.xkv_quantized_row_bytes(r, bits)), dtype=torch.uint8, device="cuda")
            xb.xkv_quantize_rows(dev[n], batch * L, r, A[n], bits=bits)
            for b in seqs:
                x = oracle.dequantize_rows(*oracle.quantize_rows(case[n][b], bits))
                hat[n][b] = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x.astype(np.float32))).astype(np.float64)
    idx_d = torch.from_numpy(idx).cuda()
    for use_counts in (False, True):
        cnt = torch.from_numpy(counts).cuda() if use_counts else None
        if bits:
            xb.xkv_gather_attend_q(shape, layer, A["A_k"], A["A_v"], bits, dev["B_k"], dev["B_v"], q, idx_d, cnt, 0.0, out, ws)
        else:
            xb.xkv_gather_attend_ex(shape, layer, A["A_k"], A["A_v"], dev["B_k"], dev["B_v"], q, idx_d, cnt, 0.0, out, ws)
        torch.cuda.synchronize()
        got = synth.storage_to_f64(synth.to_host(out))
        for b in seqs:
            rows = [idx[b, g, :(counts[b, g] if use_counts else k)] for g in range(H_kv)]
            ref, mag = reference(hat["A_k"][b], hat["A_v"][b], synth.storage_to_f64(case["B_k"][b, layer]),
                                 synth.storage_to_f64(case["B_v"][b, layer]), synth.storage_to_f64(case["q"][layer, b]), rows,
                                 oracle.default_scale(128))
            if r_v > 768:  # (the other kernel rounds the reconstructed rows as well: the tolerance of its own tests)
                assert np.abs(got[b] - ref).max() <= 2e-2 * max(np.abs(ref).max(), 1e-30)
                continue
            bound = 1.05 * 2.0 ** -8 * (np.abs(ref) + mag) + 1e-6 * np.abs(mag).max()
            over = np.abs(got[b] - ref) - bound
            assert over.max() <= 0, (b, float(over.max()), float(np.abs(got[b] - ref).max()), float(mag.max()))


def test_a_million_selected_rows_and_a_tail():
    """One KV head, every token of a long context selected: as many splits as the merge takes beside the tail's partials."""
    torch = torch_mod()
    L, r, T = 1 << 20, 16, 5
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    A_k, A_v, B_k, B_v, q = rnd(1, L, r), rnd(1, L, r), rnd(1, 1, r, 128), rnd(1, 1, r, 128), rnd(1, 1, 128)
    K_t, V_t = rnd(1, 1, T, 128), rnd(1, 1, T, 128)
    shape = xb.Shape(G=1, H_kv=1, H_q=1, d_h=128, r_k=r, r_v=r, L=L, k=L, batch=1)
    out = torch.empty((1, 1, 128), dtype=torch.bfloat16, device="cuda")
    xb.xkv_sr_decode_tail(shape, 0, A_k, A_v, B_k, B_v, q, K_t, V_t, T, out, None, None, xb.alloc_workspace(shape))
    torch.cuda.synchronize()
    K = torch.cat([A_k[0].double() @ B_k[0, 0].double(), K_t[0, 0].double()])
    V = torch.cat([A_v[0].double() @ B_v[0, 0].double(), V_t[0, 0].double()])
    w = torch.softmax(K @ q[0, 0].double() / 128 ** 0.5, 0)
    ref, mag = w @ V, w @ V.abs()
    bound = 1.05 * 2.0 ** -8 * (ref.abs() + mag) + 1e-6 * mag.max()
    assert ((out[0, 0].double() - ref).abs() <= bound).all(), float(((out[0, 0].double() - ref).abs() - bound).max())


# (H_kv, n_rep, r_k, r_v, batch): batch H_kv ceil(r_k / 128) 4 wavefronts, from 512 of them on one projection of the queries serves
# the scores and the selected rows.  Both sides of that, rank counts that end within a fragment, within 8 fragments and at 1024, 2 to
# 16 query heads per KV head and one, which keeps two projections
ONE_PROJECTION = [(8, 4, 512, 512, 4), (8, 4, 512, 512, 3), (3, 5, 144, 256, 22), (1, 16, 80, 16, 128), (2, 9, 1024, 768, 8), (5, 2, 272, 640, 9), (8, 1, 256, 128, 8)]


@pytest.mark.parametrize("H_kv,n_rep,r_k,r_v,batch", ONE_PROJECTION)
def test_whole_step_equals_its_stages(H_kv, n_rep, r_k, r_v, batch):
    """The step (B_l packed once, and in its plain layout) against the stage call on its selection, bit for bit: the projected
    queries come from the launch that projects them for the scores in the first two, from one of their own in the third."""
    torch = torch_mod()
    L, k = 300, 40
    gen = torch.Generator(device="cuda").manual_seed(r_k + r_v)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    A_k, A_v, B_k, B_v = rnd(batch, L, r_k), rnd(batch, L, r_v), rnd(batch, 2, r_k, H_kv * 128), rnd(batch, 2, r_v, H_kv * 128)
    q = rnd(batch, H_kv * n_rep, 128) * 0.05
    shape = xb.Shape(G=2, H_kv=H_kv, H_q=H_kv * n_rep, d_h=128, r_k=r_k, r_v=r_v, L=L, k=k, batch=batch)
    packed = torch.empty(xb.xkv_packed_b_bytes(shape), dtype=torch.uint8, device="cuda")
    xb.xkv_pack_b(shape, B_k, B_v, packed)
    ws = xb.alloc_workspace(shape)
    idx = torch.empty((batch, H_kv, k), dtype=torch.int32, device="cuda")
    got = []
    for call in (lambda out: xb.xkv_sr_decode_packed(shape, 1, A_k, A_v, B_k, packed, q, out, idx, None, ws),
                 lambda out: xb.xkv_sr_decode(shape, 1, A_k, A_v, B_k, B_v, q, out, idx, None, ws),
                 lambda out: xb.xkv_gather_attend(shape, 1, A_k, A_v, B_k, B_v, q, idx, out, ws)):
        ws.fill_(0xFF)                         # nothing may be left over from the call before
        got.append(torch.full((batch, H_kv * n_rep, 128), float("nan"), dtype=torch.bfloat16, device="cuda"))
        call(got[-1])
        torch.cuda.synchronize()
    assert torch.isfinite(got[2]).all() and torch.equal(got[0], got[2]) and torch.equal(got[1], got[2])

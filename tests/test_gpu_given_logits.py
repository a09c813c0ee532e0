"""Row sums from given logits: the absorbed step's attention and the second half of the step on rotated rows.  Query heads per KV head
at the edges of their copies, ranks at the edges of the groups, lists shorter and longer than a tile, quantised rows."""
import numpy as np
import pytest

from paper_2503_18893_amd import synth
from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


def torch_mod():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def rows_of(torch, A, bits):
    """What the step reads (A itself or its quantised rows), and the same in double precision."""
    if bits == 0:
        return A, A.double()
    b, L, r = A.shape
    q = torch.empty((b, L, xb.xkv_quantized_row_bytes(r, bits)), dtype=torch.uint8, device="cuda")
    xb.xkv_quantize_rows(A, b * L, r, q, bits)
    g = A.double().view(b, L, r // 32, 32)
    lo, hi = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    n = (1 << bits) - 1
    step = ((hi - lo).float() / n).bfloat16().float()
    step = torch.where(step > 0, step, torch.ones_like(step))
    codes = ((g.float() - lo.float()) * (1.0 / step)).round().clamp(0, n)
    return q, (step.double() * codes.double() + lo).view(b, L, r)


def workload(H_kv, n_rep, r_k, r_v, L, k, batch):
    return synth.Workload("given_logits", G=1, H_kv=H_kv, H_q=H_kv * n_rep, d_h=128, r_k=r_k, r_v=r_v, L=L, k=k, batch=batch,
                          dtype="bf16", a_scale=1.0, sigma_decay=0.5, q_scale=0.3)


# query heads per KV head, r_v, L, k, batch of the absorbed step; the first two are summed by the general kernels
CASES = [(1, 32, 300, 1, 1), (2, 96, 900, 127, 2), (3, 32, 300, 1, 1), (1, 32, 2500, 1025, 1), (2, 96, 1300, 1151, 2), (4, 512, 3000, 1000, 2),
         (5, 384, 700, 129, 1), (7, 640, 2000, 600, 1), (8, 256, 1000, 1000, 3), (12, 768, 900, 400, 1), (16, 128, 5000, 4500, 1)]
CASES_H_KV = 3


@pytest.mark.parametrize("bits", [0, 4])
@pytest.mark.parametrize("n_rep,r_v,L,k,batch", CASES)
def test_attention_from_kept_scores(n_rep, r_v, L, k, batch, bits):
    torch = torch_mod()
    H_kv = CASES_H_KV
    w = workload(H_kv, n_rep, 64, r_v, L, k, batch)
    g = torch.Generator(device="cuda").manual_seed(L + r_v + bits)
    A_v = torch.randn((batch, L, r_v), generator=g, device="cuda").bfloat16()
    B_v = (torch.randn((batch, 1, r_v, H_kv * 128), generator=g, device="cuda") / r_v ** 0.5).bfloat16()
    pitch = 1 << (n_rep - 1).bit_length()
    heads = torch.randn((batch, H_kv, L, pitch), generator=g, device="cuda") * 3
    idx = torch.stack([torch.randperm(L, generator=g, device="cuda")[:k].sort().values for _ in range(batch * H_kv)])
    idx = idx.view(batch, H_kv, k).int().contiguous()
    given, A64 = rows_of(torch, A_v, bits)
    shape = xb.Shape.of(w)
    ws = torch.empty(xb.xkv_absorbed_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    out = torch.empty((batch, H_kv * n_rep, 128), dtype=torch.bfloat16, device="cuda")
    (xb.xkv_attend_absorbed_q4 if bits else xb.xkv_attend_absorbed)(shape, 0, given, B_v, heads, idx, out, ws)
    for b in range(batch):
        for h in range(H_kv):
            t = idx[b, h].long()
            W = torch.softmax(heads[b, h, t, :n_rep].double(), 0)
            ref = (W.T @ A64[b, t]) @ B_v[b, 0, :, h * 128:(h + 1) * 128].double()
            got = out[b, h * n_rep:(h + 1) * n_rep].double()
            # single-precision sums (weights and sums split into 16 bits and more), one rounding to the 8 bits of bf16: at most
            # 2^-8 of the value, half a unit of its last place where it is just above a power of two
            assert (got - ref).abs().max() <= (2.0 ** -8 + 2.0 ** -13) * ref.abs().max() + 1e-6, (b, h)


@pytest.mark.parametrize("bits", [0, 4])
@pytest.mark.parametrize("what", ["sums", "weights"])
@pytest.mark.parametrize("n_rep,r_v,L,k,batch", [(1, 64, 300, 96, 2), (3, 64, 300, 96, 2), (4, 96, 300, 96, 2), (8, 128, 400, 200, 1), (7, 384, 700, 300, 1),
                                                 (12, 512, 300, 96, 1), (16, 768, 700, 300, 1)])
def test_sums_keep_single_precision(n_rep, r_v, L, k, batch, what, bits):
    """Outputs in which almost everything cancels, so that the rounding to bf16 at the end does not hide what came before it."""
    torch = torch_mod()
    H_kv = 2
    shape = xb.Shape.of(workload(H_kv, n_rep, 64, r_v, L, k, batch))
    g = torch.Generator(device="cuda").manual_seed(L + r_v + bits)
    A_v = torch.randn((batch, L, r_v), generator=g, device="cuda").bfloat16()
    pitch = 1 << (n_rep - 1).bit_length()
    heads = torch.randn((batch, H_kv, L, pitch), generator=g, device="cuda")
    B_v = torch.zeros((batch, 1, r_v, H_kv * 128), device="cuda")
    B_v[:, 0, 0] = torch.rand((H_kv * 128,), generator=g, device="cuda") + 0.5
    if what == "sums":  # of two columns that differ only in rows of little weight, the difference
        A_v[:, :, 0] = (torch.rand((batch, L), generator=g, device="cuda") + 0.5).bfloat16()
        A_v[:, :, 1] = A_v[:, :, 0]
        A_v[:, ::10, 1] = 1 - A_v[:, ::10, 0]
        heads[:, :, ::10] -= 9.0
        B_v[:, 0, 1] = -B_v[:, 0, 0]
        pick, group = L, 1
    else:  # rows in pairs of opposite sign and nearly equal weight
        A_v = A_v.clamp(-1, 1)
        A_v[:, 0::2, 0], A_v[:, 1::2, 0] = 1, -1
        heads[:, :, 1::2] = heads[:, :, 0::2] + 1e-4 * torch.randn((batch, H_kv, L // 2, pitch), generator=g, device="cuda")
        pick, group = L // 2, 2
    B_v = B_v.bfloat16()
    idx = torch.stack([torch.randperm(pick, generator=g, device="cuda")[:k // group].sort().values for _ in range(batch * H_kv)])
    idx = (group * idx[:, :, None] + torch.arange(group, device="cuda")).view(batch, H_kv, k).int().contiguous()
    given, A64 = rows_of(torch, A_v, bits)
    ws = torch.empty(xb.xkv_absorbed_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    out = torch.empty((batch, H_kv * n_rep, 128), dtype=torch.bfloat16, device="cuda")
    (xb.xkv_attend_absorbed_q4 if bits else xb.xkv_attend_absorbed)(shape, 0, given, B_v, heads, idx, out, ws)
    for b in range(batch):
        for h in range(H_kv):
            t = idx[b, h].long()
            W = torch.softmax(heads[b, h, t, :n_rep].double(), 0)
            B64 = B_v[b, 0, :, h * 128:(h + 1) * 128].double()
            ref, size = (W.T @ A64[b, t]) @ B64, (W.T @ A64[b, t].abs()) @ B64.abs()
            err = ((out[b, h * n_rep:(h + 1) * n_rep].double() - ref).abs() - 2.0 ** -8 * ref.abs()).clamp_min(0)
            # sums of 300 products or fewer, each rounded to 24 bits of a partial sum: a few units of the last place of the whole
            # (rounding errors that add up at random: sqrt(300) halves are 9); weights within two units, over rows that do not add up
            assert (err / size).max() <= (8 if what == "sums" else 2) * 2.0 ** -24, (b, h)


# bits, query heads per KV head (8 of them), ranks, k, batch: all in two halves.  The logits take the room of the projected queries and
# the scores, so the context is as long as they are.
ROTATED = [(0, 4, 64, 12300, 2), (0, 7, 96, 12300, 2), (0, 8, 320, 12300, 2), (0, 1, 512, 4100, 6), (0, 3, 448, 4100, 6), (0, 4, 256, 9300, 8),
           (4, 4, 64, 12300, 2), (4, 7, 160, 20500, 2), (4, 1, 512, 8200, 2), (4, 3, 288, 8200, 2), (4, 8, 384, 12300, 2),
           (3, 4, 64, 12300, 2), (3, 2, 512, 8200, 2), (3, 6, 512, 12300, 2)]


def rotated_shape(n_rep, r, k, batch):
    return dict(H_kv=8, H_q=8 * n_rep, r_k=r, r_v=r, L=k << (n_rep - 1).bit_length(), k=k, batch=batch)


@pytest.mark.parametrize("bits,n_rep,r,k,batch", ROTATED)
def test_rotated_rows_in_two_halves(bits, n_rep, r, k, batch):
    torch = torch_mod()
    f = rotated_shape(n_rep, r, k, batch)
    H_kv, L, theta = f["H_kv"], f["L"], 500000.0
    shape = xb.Shape(G=1, d_h=128, dtype="bf16", **f)
    g = torch.Generator(device="cuda").manual_seed(r + bits)
    A = [torch.randn((batch, L, r), generator=g, device="cuda").bfloat16() for _ in "kv"]
    B = [(torch.randn((batch, 1, r, H_kv * 128), generator=g, device="cuda") / r ** 0.5).bfloat16() for _ in "kv"]
    q = torch.randn((batch, H_kv * n_rep, 128), generator=g, device="cuda").bfloat16()
    idx = torch.stack([torch.randperm(L, generator=g, device="cuda")[:k].sort().values for _ in range(batch * H_kv)])
    idx = idx.view(batch, H_kv, k).int().contiguous()
    counts = torch.full((batch, H_kv), k, dtype=torch.int32, device="cuda")
    counts[0, 1], counts[1, 2], counts[1, 3] = 1, 4097, 0
    given = [rows_of(torch, a, bits) for a in A]
    ws = xb.alloc_workspace(shape)
    out = torch.empty_like(q)
    if bits:
        xb.xkv_gather_attend_q(shape, 0, given[0][0], given[1][0], bits, B[0], B[1], q, idx, counts, theta, out, ws)
    else:
        xb.xkv_gather_attend_ex(shape, 0, A[0], A[1], B[0], B[1], q, idx, counts, theta, out, ws)
    freq = theta ** (-torch.arange(64, device="cuda", dtype=torch.float64) / 64)
    for b in range(batch):
        for h in range(H_kv):
            n = int(counts[b, h])
            t = idx[b, h, :n].long()
            got = out[b, h * n_rep:(h + 1) * n_rep].double()
            if n == 0:
                assert (got == 0).all()
                continue
            # keys as the kernel has them: rows in bf16, rotated, in bf16 again; from there on everything is exact but for 2^-16 of a
            # weight, single-precision angles and sums (the few keys that these round the other way) and the last rounding
            K = given[0][1][b, t].bfloat16().double() @ B[0][b, 0, :, h * 128:(h + 1) * 128].double()
            c, s = (t[:, None] * freq).cos(), (t[:, None] * freq).sin()
            K = torch.cat((K[:, :64] * c - K[:, 64:] * s, K[:, 64:] * c + K[:, :64] * s), 1).bfloat16().double()
            W = torch.softmax(K @ q[b, h * n_rep:(h + 1) * n_rep].double().T / 128 ** 0.5, 0)
            ref = W.T @ (given[1][1][b, t] @ B[1][b, 0, :, h * 128:(h + 1) * 128].double())
            err, size = (got - ref).square().mean().sqrt(), ref.square().mean().sqrt()
            assert err <= 2.0 ** -8 * size, (b, h)  # (twice what the last rounding alone can be)

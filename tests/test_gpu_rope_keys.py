"""Rotated rows in two halves where the keys' factor stays in registers (ranks up to 512, up to eight query heads per KV head), at the
edges of its tiles of 32 rows and runs, and the other form of the same (more ranks of the keys than of the values)."""
import pytest

from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


CASES = [
    (0, 4, 128, 128, 1025, 32), (0, 8, 512, 64, 1057, 32), (0, 1, 80, 48, 2049, 16), (0, 4, 384, 512, 1031, 32), (0, 2, 640, 256, 8200, 6),
    (4, 8, 512, 512, 1025, 32), (4, 4, 32, 64, 1056, 32), (4, 5, 352, 384, 1023, 33), (4, 4, 640, 512, 8200, 2), (3, 4, 256, 256, 1025, 32), (3, 8, 480, 96, 1025, 32),
    (3, 4, 352, 128, 1025, 32), (3, 4, 640, 512, 8200, 2)]


def shape_of(n_rep, r_k, r_v, k, batch):  # (the logits' room is the scores')
    return dict(G=1, H_kv=8, H_q=8 * n_rep, d_h=128, r_k=r_k, r_v=r_v, L=k << (n_rep - 1).bit_length(), k=k, batch=batch)


@pytest.mark.parametrize("bits,n_rep,r_k,r_v,k,batch", CASES)
def test_rotated_rows(bits, n_rep, r_k, r_v, k, batch):
    check(bits, n_rep, r_k, r_v, k, batch)


@pytest.mark.parametrize("bits,r_k", [(4, 512), (4, 96), (3, 352)])
def test_steps_up_to_the_end_of_the_range(bits, r_k):
    """Groups of 32 ranks whose steps (0.2 to 0.7 of the powers) lie on both sides of 2^104, up to 2^120; the factor's rows are as much smaller."""
    check(bits, 4, r_k, 64, 1025, 32, powers=[0, 106, 121, 104, 105, 1, 110, 118, 102])


def check(bits, n_rep, r_k, r_v, k, batch, powers=None):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = shape_of(n_rep, r_k, r_v, k, batch)
    H_kv, theta, L = f["H_kv"], 500000.0, f["L"]
    shape = xb.Shape(dtype="bf16", **f)
    g = torch.Generator(device="cuda").manual_seed(r_k + bits)
    A = [torch.randn((batch, L, r), generator=g, device="cuda").bfloat16() for r in (r_k, r_v)]
    B = [(torch.randn((batch, 1, r, H_kv * 128), generator=g, device="cuda") / r ** 0.5).bfloat16() for r in (r_k, r_v)]
    if powers:  # (no element of the factor below the normal numbers)
        e = torch.tensor([powers[j // 32 % len(powers)] for j in range(r_k)], device="cuda", dtype=torch.float64)
        A[0] = (A[0].double() * 2.0 ** e).bfloat16()
        sign = 2.0 * torch.randint(0, 2, B[0].shape, generator=g, device="cuda") - 1
        B[0] = (sign * (0.5 + 0.5 * torch.rand(B[0].shape, generator=g, device="cuda")) * 2.0 ** -(e[:, None] + 4)).bfloat16()
    q = torch.randn((batch, H_kv * n_rep, 128), generator=g, device="cuda").bfloat16()
    idx = torch.argsort(torch.rand((batch, H_kv, L), generator=g, device="cuda"), dim=-1)[..., :k].sort(-1).values.int().contiguous()
    counts = torch.full((batch, H_kv), k, dtype=torch.int32, device="cuda")
    counts[0, 1], counts[0, 2], counts[1, 0], counts[1, 3] = 1, 33, 0, k - 1
    ws = torch.full((xb.xkv_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")  # NaN where nothing is written
    out = torch.empty_like(q)
    rows = rows_of(A, bits)
    if bits:
        xb.xkv_gather_attend_q(shape, 0, rows[0], rows[1], bits, B[0], B[1], q, idx, counts, theta, out, ws)
    else:
        xb.xkv_gather_attend_ex(shape, 0, rows[0], rows[1], B[0], B[1], q, idx, counts, theta, out, ws)
    compare(A, bits, [b[:, 0] for b in B], q, idx, counts, theta, out)


def rows_of(A, bits):
    """A^K and A^V as the calls take them."""
    import torch
    if not bits:
        return A
    rows = []
    for a in A:
        n, r = a.shape[0] * a.shape[1], a.shape[2]
        rows.append(torch.empty((n, xb.xkv_quantized_row_bytes(r, bits)), dtype=torch.uint8, device="cuda"))
        xb.xkv_quantize_rows(a, n, r, rows[-1], bits)
    return rows


def levels(a, bits):
    """What rows of A hold, in double precision."""
    import torch
    if not bits:
        return a.double()
    v, top = a.float().unflatten(-1, (-1, 32)), 2.0 ** bits - 1
    lo, hi = v.amin(-1, keepdim=True), v.amax(-1, keepdim=True)
    step = ((hi - lo) / top).bfloat16().float()
    step = torch.where(step == 0, torch.ones_like(step), step)
    return (step.double() * ((v - lo) * (1.0 / step)).round().clamp(0, top).double() + lo.double()).flatten(-2)


def compare(A, bits, B, q, idx, counts, theta, out):
    """`out` for some KV heads of the first two and the last sequence.  B: one layer's, [batch][rank][H_kv * 128]."""
    import torch
    batch, H_kv = counts.shape
    n_rep = q.shape[1] // H_kv
    freq = theta ** (-torch.arange(64, device="cuda", dtype=torch.float64) / 64)
    for b, h in [(0, 0), (0, 1), (0, 2), (1, 0), (1, 3), (batch - 1, H_kv - 1)]:
        t = idx[b, h, :int(counts[b, h])].long()
        got = out[b, h * n_rep:(h + 1) * n_rep].double()
        if len(t) == 0:
            assert (got == 0).all()
            continue
        # keys as the kernel has them: rows in bf16, rotated, in bf16 again; what is left are 2^-16 of a weight, single-precision angles and
        # sums (the few keys that these round the other way) and the last rounding, 2^-9 of a value at most
        cols = slice(h * 128, (h + 1) * 128)
        K = levels(A[0][b, t], bits).bfloat16().double() @ B[0][b, :, cols].double()
        c, s = (t[:, None] * freq).cos(), (t[:, None] * freq).sin()
        K = torch.cat((K[:, :64] * c - K[:, 64:] * s, K[:, 64:] * c + K[:, :64] * s), 1).bfloat16().double()
        W = torch.softmax(K @ q[b, h * n_rep:(h + 1) * n_rep].double().T / 128 ** 0.5, 0)
        ref = W.T @ (levels(A[1][b, t], bits) @ B[1][b, :, cols].double())
        err, size = (got - ref).square().mean().sqrt(), ref.square().mean().sqrt()
        assert err <= 2.0 ** -8 * size, (b, h)  # (twice what the last rounding alone can be)


LAYERS = dict(G=3, H_kv=8, H_q=32, d_h=128, r_k=256, r_v=96, L=4203, k=1001, batch=32)  # with c = 8 and o = 3: 1032 rows


@pytest.mark.parametrize("bits", [0, 4])
def test_last_layer_of_a_packed_group(bits):
    """The landmark step on the factor as xkv_pack_b leaves it, several sequences and layers: the same bits as on the plain one."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f, c, o, theta = LAYERS, 8, 3, 500000.0
    G, H_kv, batch, L, cap, layer = f["G"], f["H_kv"], f["batch"], f["L"], 1032, f["G"] - 1
    shape, n_c = xb.Shape(dtype="bf16", **f), -(-f["L"] // c)
    g = torch.Generator(device="cuda").manual_seed(7 + bits)
    A = [torch.randn((batch, L, f[r]), generator=g, device="cuda").bfloat16() for r in ("r_k", "r_v")]
    B = [(torch.randn((batch, G, f[r], H_kv * 128), generator=g, device="cuda") / f[r] ** 0.5).bfloat16() for r in ("r_k", "r_v")]
    q = torch.randn((batch, f["H_q"], 128), generator=g, device="cuda").bfloat16()
    marks = torch.randn((batch, H_kv, n_c, 128), generator=g, device="cuda").bfloat16()
    outliers = torch.argsort(torch.rand((batch, H_kv, n_c), generator=g, device="cuda"), -1)[..., :o].sort(-1).values.int().contiguous()
    packed = torch.empty(xb.xkv_packed_b_bytes(shape), dtype=torch.uint8, device="cuda")
    xb.xkv_pack_b(shape, B[0], B[1], packed)
    rows, results = rows_of(A, bits), []
    for form in ("plain", "packed"):
        ws = torch.full((xb.xkv_landmark_workspace_bytes(shape, c, o),), 255, dtype=torch.uint8, device="cuda")
        out, ids = torch.empty_like(q), torch.zeros((batch, H_kv, cap), dtype=torch.int32, device="cuda")
        counts = torch.empty((batch, H_kv), dtype=torch.int32, device="cuda")
        rest = (q, marks, outliers, c, o, out, ids, counts, None, ws)
        if form == "packed":
            xb.xkv_sr_decode_landmark_packed(shape, layer, *rows, bits, B[0], packed, *rest, rope_theta=theta)
        elif bits:
            xb.xkv_sr_decode_landmark_q(shape, layer, *rows, bits, *B, *rest, rope_theta=theta)
        else:
            xb.xkv_sr_decode_landmark(shape, layer, *rows, *B, *rest, rope_theta=theta)
        results.append((out, ids, counts))
    (out, ids, counts), (plain_out, _, plain_counts) = results[1], results[0]
    assert torch.equal(out, plain_out) and torch.equal(counts, plain_counts)
    assert (counts >= f["k"] - c).all() and (counts <= cap).all()
    compare(A, bits, [b[:, layer] for b in B], q, ids, counts, theta, out)

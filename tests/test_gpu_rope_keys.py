"""Rotated rows in two halves where the keys' factor stays in registers (ranks up to 512, up to eight query heads per KV head), at the
edges of its tiles of 32 rows and runs, and the other form of the same (more ranks of the keys than of the values)."""
import pytest

from paper_2503_18893_amd import binding as xb

pytestmark = pytest.mark.gpu


CASES = [
    (0, 4, 128, 128, 1025, 32), (0, 8, 512, 64, 1057, 32), (0, 1, 80, 48, 2049, 16), (0, 4, 384, 512, 1031, 32), (0, 2, 640, 256, 8200, 6),
    (4, 8, 512, 512, 1025, 32), (4, 4, 32, 64, 1056, 32), (4, 5, 352, 384, 1023, 33), (4, 4, 640, 512, 8200, 2), (3, 4, 256, 256, 1025, 32), (3, 8, 480, 96, 1025, 32)]


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
    H_kv, theta, L = 8, 500000.0, k << (n_rep - 1).bit_length()
    shape = xb.Shape(G=1, H_kv=H_kv, H_q=H_kv * n_rep, d_h=128, r_k=r_k, r_v=r_v, L=L, k=k, batch=batch, dtype="bf16")
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
    rows = A
    if bits:
        rows = []
        for a in A:
            rows.append(torch.empty((batch * L, xb.xkv_quantized_row_bytes(a.shape[-1], bits)), dtype=torch.uint8, device="cuda"))
            xb.xkv_quantize_rows(a, batch * L, a.shape[-1], rows[-1], bits)
        xb.xkv_gather_attend_q(shape, 0, rows[0], rows[1], bits, B[0], B[1], q, idx, counts, theta, out, ws)
    else:
        xb.xkv_gather_attend_ex(shape, 0, rows[0], rows[1], B[0], B[1], q, idx, counts, theta, out, ws)

    def levels(a):  # what quantised rows hold
        if not bits:
            return a.double()
        v, top = a.float().unflatten(-1, (-1, 32)), 2.0 ** bits - 1
        lo, hi = v.amin(-1, keepdim=True), v.amax(-1, keepdim=True)
        step = ((hi - lo) / top).bfloat16().float()
        step = torch.where(step == 0, torch.ones_like(step), step)
        return (step.double() * ((v - lo) * (1.0 / step)).round().clamp(0, top).double() + lo.double()).flatten(-2)

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
        K = levels(A[0][b, t]).bfloat16().double() @ B[0][b, 0, :, cols].double()
        c, s = (t[:, None] * freq).cos(), (t[:, None] * freq).sin()
        K = torch.cat((K[:, :64] * c - K[:, 64:] * s, K[:, 64:] * c + K[:, :64] * s), 1).bfloat16().double()
        W = torch.softmax(K @ q[b, h * n_rep:(h + 1) * n_rep].double().T / 128 ** 0.5, 0)
        ref = W.T @ (levels(A[1][b, t]) @ B[1][b, 0, :, cols].double())
        err, size = (got - ref).square().mean().sqrt(), ref.square().mean().sqrt()
        assert err <= 2.0 ** -8 * size, (b, h)  # (twice what the last rounding alone can be)

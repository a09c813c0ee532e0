"""The once-per-prompt kernels where their work is cut: quantised rows shorter and longer than a workgroup's share, steps
outside the range of the short quotient, landmark chunks of 4 to 16 keys that do not fill a wavefront or the last chunk."""
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


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("rows,r", [(257, 32), (11, 800), (5, 2048), (5, 2080), (3, 8192), (5, 8224), (130, 4128), (393217, 32), (12300, 1056), (192, 65568)])
def test_quantised_rows_at_the_edges_of_a_workgroup(rows, r, bits):
    torch = torch_mod()
    rng = np.random.default_rng(rows + r)
    x = rng.standard_normal((rows, r))
    x[0, :32] *= 1e-30                   # steps below and above the range of the short quotient
    x[rows - 1, r - 32:] *= 1e30
    x[1, :32] = -0.0
    xbits = synth.to_storage(x, "bf16")
    X = torch.from_numpy(xbits.view(np.int16)).cuda()
    pitch = xb.xkv_quantized_row_bytes(r, bits)
    out = torch.full((rows + 1, pitch), 0xAB, dtype=torch.uint8, device="cuda")
    xb.xkv_quantize_rows(X, rows, r, out, bits)
    got = out.cpu().numpy()
    codes, step, lo = oracle.quantize_rows(xbits, bits)
    want = (oracle.pack_q4 if bits == 4 else oracle.pack_q3)(codes, step, lo)
    np.testing.assert_array_equal(got[:rows], want)
    assert (got[rows] == 0xAB).all()     # nothing behind the last row


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("rows,r", [(4096, 512), (4097, 512), (260, 8192), (259, 8224), (9363, 224), (21846, 96), (65537, 32),
                                    (65537, 256), (4081, 4128), (2041, 8224), (5120, 512), (5121, 512), (321, 8192), (319, 8224),
                                    (11703, 224), (27307, 96), (81921, 32), (6656, 512), (6657, 512), (417, 8192), (15213, 224), (15214, 224)])
def test_quantised_rows_a_lane_per_group(rows, r, bits):
    """Both sides of 416 x 1024 pieces; 256 groups a row, one more, and numbers of groups that do not divide a workgroup; more than 2^21
    pieces."""
    test_quantised_rows_at_the_edges_of_a_workgroup(rows, r, bits)


@pytest.mark.parametrize("bits,rows,r", [(4, 524289, 512), (3, 655361, 512), (4, 163900, 1632)])
def test_packed_rows_beyond_the_caches(bits, rows, r):
    """More than 160 MiB of packed rows, the last workgroup not full: the same bytes as from calls of a tenth."""
    torch = torch_mod()
    X = torch.randn((rows, r), generator=torch.Generator(device="cuda").manual_seed(rows), device="cuda", dtype=torch.bfloat16)
    pitch = xb.xkv_quantized_row_bytes(r, bits)
    out = torch.full((rows + 1, pitch), 0xAB, dtype=torch.uint8, device="cuda")
    xb.xkv_quantize_rows(X, rows, r, out, bits)
    assert rows * pitch > 160 << 20
    step = rows // 10
    for first in range(0, rows, step):
        n = min(step, rows - first)
        part = torch.empty((n, pitch), dtype=torch.uint8, device="cuda")
        xb.xkv_quantize_rows(X[first:], n, r, part, bits)
        assert torch.equal(out[first:first + n], part), first
    assert bool((out[rows] == 0xAB).all())


@pytest.mark.parametrize("c", [4, 8, 12, 16])
@pytest.mark.parametrize("chunks,rest", [(1, 0), (15, 1), (16, 0), (17, 3), (64, 2)])
def test_landmarks_at_the_edges_of_a_wavefront(c, chunks, rest):
    torch = torch_mod()
    L = chunks * c + rest
    w = synth.Workload("landmark_edges", G=1, H_kv=2, H_q=4, d_h=128, r_k=16, r_v=16, L=L, k=1, batch=2, dtype="bf16",
                       a_scale=1.0, sigma_decay=0.5, q_scale=0.3)
    K = synth.to_storage(np.random.default_rng(L + c).standard_normal((2, 2, L, 128)) + 0.5, "bf16")
    K[1, 1, L - 1] = 0                   # a zero key counts as cosine 0
    n_c = -(-L // c)
    shape = xb.Shape.of(w)
    Lm = torch.zeros((2, 2, n_c, 128), dtype=torch.bfloat16, device="cuda")
    negm = torch.full((2, 2, n_c), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.empty(xb.xkv_landmark_workspace_bytes(shape, c, 0), dtype=torch.uint8, device="cuda")
    xb.xkv_landmarks(shape, synth.to_device({"K": K}, "bf16")["K"], c, 0, Lm, negm, None, ws)
    got, m = synth.storage_to_f64(synth.to_host(Lm)), negm.cpu().numpy().astype(np.float64)
    for b in range(2):
        ref, m_ref, _ = oracle.landmarks(K[b], c, 0)
        # one rounding to bf16; a cosine of two sums of 128 products in single precision
        assert np.abs(got[b] - ref).max() <= 2.0 ** -8 * np.abs(ref).max()
        assert np.abs(-m[b] - m_ref).max() <= 128 * 2.0 ** -23

"""How a shape is split over workgroups (make_plan, host code): the limits that the launches rely on.  No GPU needed."""
import os
import subprocess

import pytest

from paper_2503_18893_amd import build as xbuild
from test_gpu_gather_absorb import CASES
import test_gpu_given_logits as given
import test_gpu_reconstruct_tiles as tiles
import test_gpu_rope_keys as rope


@pytest.fixture(scope="module")
def plan_of(tmp_path_factory):
    """Plans of a list of dicts with the shape's fields (the rest: one layer of the Llama shape)."""
    objs = [os.path.join(xbuild.OBJ_DIR, src.replace(".hip", ".o")) for src in xbuild.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        xbuild.build_library()
    exe = str(tmp_path_factory.mktemp("plan") / "probe")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "plan_probe.cpp")
    subprocess.run([xbuild._hipcc(), *xbuild.HIPCC_FLAGS, "-x", "hip", src, "-x", "none", *objs, "-o", exe], check=True,
                   capture_output=True)

    def run(shapes):
        base = dict(G=1, H_kv=8, H_q=32, d_h=128, r_k=512, r_v=512, L=1, k=1, batch=1, dtype=1)
        lines = []
        for sh in shapes:
            f = {**base, **sh}
            f["L"] = max(f["L"], f["k"])
            lines.append(" ".join(str(f[n]) for n in base))
        out = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(shapes)
        return [{n: int(v) for n, v in (kv.split("=") for kv in line.split())} for line in out]
    return run


def test_partials_of_a_step_fit_the_merge(plan_of):
    """Selected rows and uncompressed tail together, wherever the limit of 4096 rows per workgroup leaves room for both."""
    shapes = [dict(H_kv=h, H_q=h, batch=b, r_k=r, r_v=r, k=k) for h, b in ((1, 1), (2, 1), (1, 3), (8, 1), (8, 5))
              for r in (16, 384) for k in (1, 129, 4097, 100_000, 500_000, 1 << 20, (1 << 20) + 1, 3_000_000, 992 * 4096)]
    for sh, p in zip(shapes, plan_of(shapes)):
        assert p["absorb"] == 1 and p["splits"] * p["chunk"] >= sh["k"] > (p["splits"] - 1) * p["chunk"], (sh, p)
        assert p["splits"] + p["tail_parts"] <= p["merge_limit"] and p["splits"] <= p["max_splits"], (sh, p)


def test_workgroups_per_compute_unit_follow_from_the_lds(plan_of):
    """Two workgroups are counted on only where both fit, and one round of workgroups is not left for a few of a second."""
    shapes = [dict(batch=b, k=k, r_k=rk, r_v=rv) for b in (1, 2, 3, 4, 5, 6, 16) for k in (500, 2048, 4096, 16384)
              for rk in (16, 128, 384, 512, 528, 640, 768, 1024) for rv in (16, 256, 384, 512, 576, 768)]
    shared = 0
    for sh, p in zip(shapes, plan_of(shapes)):
        if not p["absorb"]:
            continue
        slots, work, tiles = 256 if p["occ"] == 1 else 1024, 8 * sh["batch"] * p["splits"], (sh["k"] + 127) // 128
        assert p["lds"] * p["occ"] <= 160 * 1024, (sh, p)
        assert p["occ"] == 1 or sh["r_v"] <= 512, (sh, p)
        shared += p["occ"] == 2
        # no cut of the lists would be done a whole round of tiles earlier
        time = -(-work // slots) * (p["chunk"] // 128 + 1)
        for per in range(1, tiles + 1):
            splits = -(-tiles // per)
            assert time <= -(-8 * sh["batch"] * splits // slots) * (per + 1) + 1, (sh, p, per)
    assert shared > 100


def test_which_shapes_keep_b_out_of_the_main_loop(plan_of):
    """r_k up to 1024, r_v up to 768, row offsets of one sequence within 32 bits -- and then the launch fits the LDS, at any head
    count and at the most ids per workgroup."""
    shapes = [dict(r_k=rk, r_v=rv, H_q=8 * n, k=k, L=L) for rk in (16, 640, 1008, 1024, 1040, 1280) for rv in (16, 512, 768, 784)
              for n in (1, 16) for k in (1, 4_000_000) for L in (1, 3_000_000, (1 << 24) - 1)]
    for sh, p in zip(shapes, plan_of(shapes)):
        L = max(sh["L"], sh["k"])
        ok = sh["r_k"] <= 1024 and sh["r_v"] <= 768 and L * max(sh["r_k"], sh["r_v"]) * 2 < 1 << 32
        assert p["absorb"] == ok, (sh, p)
        assert not ok or p["lds"] <= 160 * 1024 - 512, (sh, p)


def test_the_kernels_tests_reach_the_tiles_they_name(plan_of):
    shapes = [dict(H_kv=h, H_q=h * n, r_k=rk, r_v=rv, batch=b, k=k) for h, n, rk, rv, b, k, _, _ in CASES]
    for case, p in zip(CASES, plan_of(shapes)):
        assert (p["occ"], p["chunk"] // 128) == case[6:] and p["absorb"] == (case[6] > 0), (case, p)


def test_absorbed_step_takes_the_faster_kernels(plan_of):
    """Both sides of each line at which the row sums of the absorbed step change over to the general kernels, bf16 and 4-bit rows."""
    line = [  # n_rep, r, batch, k, matrix cores for bf16, for 4 bits
        (4, 512, 8, 4095, 1, 1), (4, 512, 8, 4096, 0, 1), (4, 512, 16, 4096, 0, 1), (4, 512, 16, 16384, 0, 0), (4, 128, 16, 4096, 1, 1),
        (4, 768, 4, 1024, 1, 1), (4, 768, 4, 2048, 0, 0), (8, 768, 4, 2048, 1, 1), (1, 512, 1, 1023, 0, 0), (1, 512, 1, 1024, 1, 1),
        (1, 512, 4, 4096, 0, 0), (1, 128, 16, 1024, 1, 1), (2, 256, 8, 4096, 0, 1), (1, 768, 1, 1024, 0, 0), (1, 768, 1, 2048, 1, 1),
        (9, 512, 16, 16384, 1, 1), (16, 768, 32, 4096, 1, 1)]
    shapes = [dict(H_q=8 * n, r_k=r, r_v=r, batch=b, k=k) for n, r, b, k, _, _ in line]
    for case, p in zip(line, plan_of(shapes)):
        assert (p["absorbed"], p["absorbed_q4"]) == case[4:], case
    shapes = [dict(H_kv=given.CASES_H_KV, H_q=given.CASES_H_KV * n, r_k=64, r_v=r, L=L, k=k, batch=b) for n, r, L, k, b in given.CASES]
    assert [(p["absorbed"], p["absorbed_q4"]) for p in plan_of(shapes)] == [(0, 0)] * 2 + [(1, 1)] * (len(shapes) - 2)


def test_rotated_rows_in_two_halves_where_that_is_faster(plan_of):
    """Both sides of the lines, the room that the logits need, and that the kernel's test reaches it in every case."""
    line = [  # n_rep, r, batch, k, two halves in bf16, 4 bits, 3 bits
        (4, 512, 4, 4096, 0, 1, 1), (4, 512, 6, 4096, 1, 1, 1), (4, 512, 16, 4096, 0, 1, 1), (4, 512, 3, 4096, 0, 0, 0), (4, 256, 5, 4096, 0, 0, 0),
        (4, 256, 8, 4096, 0, 1, 1), (4, 384, 5, 4096, 0, 1, 1), (4, 384, 8, 4096, 1, 1, 1), (4, 448, 8, 4096, 0, 1, 1), (8, 512, 5, 4096, 0, 0, 0),
        (8, 512, 8, 4096, 0, 1, 1), (8, 64, 8, 4096, 1, 0, 0), (8, 64, 10, 4096, 1, 1, 1), (4, 512, 16, 4128, 1, 1, 1), (1, 256, 16, 4128, 1, 1, 1), (9, 512, 16, 4096, 0, 0, 0), (4, 528, 16, 4096, 0, 0, 0)]
    shapes = [dict(H_q=8 * n, r_k=r, r_v=r, batch=b, k=k, L=16 * k) for n, r, b, k, _, _, _ in line]
    for case, p in zip(line, plan_of(shapes)):
        assert (p["kept_0"], p["kept_4"], p["kept_3"]) == case[4:], case
    for (bits, *case), p in zip(given.ROTATED, plan_of([given.rotated_shape(*case) for _, *case in given.ROTATED])):
        assert p[f"kept_{bits}"] == 1, (bits, case)
    # 4 logits a row: 16 k <= 4 L + 4 (2 H_q + 64) (r_k + 128) / H_kv, all in bytes
    room = (2 * 32 + 64) * (64 + 128) // 8
    for L, kept in ((4 * 12288 - room, 1), (4 * 12288 - room - 64, 0)):
        assert plan_of([dict(r_k=64, r_v=64, L=L, k=12288 + 0, batch=8)])[0]["kept_4"] == kept


def test_rotated_rows_whose_logits_come_from_the_factor_in_registers(plan_of):
    """Both sides of the limits of ranks, heads and rows."""
    line = [  # n_rep, r_k, r_v, batch, k, that kernel in bf16, 4 bits, 3 bits
        (4, 256, 256, 8, 4096, 1, 1, 1), (4, 256, 256, 8, 4095, 0, 1, 1), (8, 256, 256, 8, 4096, 1, 1, 1), (8, 256, 256, 8, 4095, 0, 0, 0),
        (4, 512, 512, 8, 4096, 1, 1, 1), (4, 528, 512, 8, 4096, 0, 0, 0), (4, 512, 512, 8, 4095, 0, 1, 1), (9, 256, 256, 16, 4096, 0, 0, 0),
        (4, 512, 528, 16, 4096, 0, 0, 0), (4, 512, 512, 6, 4096, 1, 1, 1), (4, 544, 512, 6, 4096, 0, 0, 0)]
    shapes = [dict(H_q=8 * n, r_k=rk, r_v=rv, batch=b, k=k, L=16 * k) for n, rk, rv, b, k, _, _, _ in line]
    for case, p in zip(line, plan_of(shapes)):
        assert (p["regs_0"], p["regs_4"], p["regs_3"]) == case[5:], case
    # bf16 rows of ranks 512 in one full round, few of the tokens: heads, rows, batch, tokens, that kernel
    few = [(4, 4096, 8, 98303, 1), (4, 4096, 8, 98304, 0), (8, 4096, 8, 65535, 1), (8, 4096, 8, 65536, 0), (4, 4128, 8, 131072, 1),
           (4, 5000, 8, 131072, 0), (4, 4096, 16, 131072, 1), (4, 4096, 10, 131072, 1), (8, 8192, 4, 131072, 0), (4, 8192, 4, 131072, 1)]
    for case, p in zip(few, plan_of([dict(H_q=8 * n, r_k=512, r_v=512, batch=b, k=k, L=L) for n, k, b, L, _ in few])):
        assert (p["regs_0"], p["regs_4"], p["regs_3"]) == (case[4], 1, 1), case
    assert all(p["regs_0"] for p in plan_of([dict(r_k=rk, r_v=rv, batch=8, k=4096, L=131072) for rk, rv in ((384, 512), (512, 496))]))
    for (bits, _, r_k, *_), p in zip(rope.CASES, plan_of([rope.shape_of(*case) for _, *case in rope.CASES])):
        assert (p[f"regs_{bits}"], p[f"kept_{bits}"] or p[f"regs_{bits}"]) == (int(r_k <= 512), 1), (bits, r_k)
    p = plan_of([{**rope.LAYERS, "k": 1032}])[0]
    assert p["regs_0"] and p["regs_4"]
    # the other kernel that leaves logits has eight wavefronts
    some = [dict(H_q=8 * n, r_k=rk, r_v=rv, batch=b, k=k, L=16 * k) for n in (1, 4, 8) for rk in (64, 512, 640) for rv in (64, 256, 512)
            for b in (1, 2, 8) for k in (1024, 8191, 8192, 16384, 20000)]
    assert all(p["waves"] == 8 for p in plan_of(some) if p["kept_0"] or p["kept_4"] or p["kept_3"])


def test_which_scores_are_long_streams(plan_of):
    """Which scores go to the long-stream kernel, a whole round of its wavefronts' tiles at a time; chunks of the selection's histograms
    are multiples of 256."""
    line = [  # tiles, r, batch, n_rep, taken
        (1056, 512, 1, 4, 0), (1057, 512, 1, 4, 1), (1057, 176, 1, 4, 0), (1057, 192, 1, 4, 1), (2112, 256, 1, 4, 0), (2113, 256, 1, 4, 1),
        (3, 512, 350, 4, 0), (20, 256, 64, 4, 0), (20, 512, 64, 4, 1), (1057, 512, 1, 16, 0), (3000, 512, 6, 4, 1), (16384, 64, 1, 4, 1),
        (16383, 64, 1, 4, 0), (141, 768, 16, 4, 1), (60, 128, 300, 4, 1)]
    shapes = [dict(H_q=8 * n, r_k=r, r_v=64, batch=b, L=32 * t, k=t) for t, r, b, n, _ in line]
    for case, p in zip(line, plan_of(shapes)):
        pairs = case[2] * (4 if case[3] == 16 else 1)
        assert p["stream"] == case[4], case
        if p["stream"] and not p["score_hist"]:
            waves = 8 if case[1] <= 640 else 4
            assert p["score_tpw"] == (-(-case[0] // max(256 // pairs, 1)) + waves - 1) // waves * waves, case
    hist = plan_of([dict(L=L, k=8192, batch=b) for L in (131072, 100_001, 262_145) for b in (4, 5, 16)])
    assert sum(p["score_hist"] for p in hist) > 3
    assert all(p["topk_chunk"] % 256 == 0 for p in hist) and all(p["topk_chunk"] == 32 * p["score_tpw"] for p in hist if p["score_hist"])


def test_reconstruction_keeps_the_factor_where_that_is_faster(plan_of):
    """Few long runs and every call of one sequence keep B_l in registers; many short sequences, each with a factor of its own, do not,
    above 256 ranks."""
    line = [  # KV heads, r, batch, L, kept
        (8, 512, 1, 32768, 1), (8, 768, 1, 64, 1), (8, 384, 4, 65536, 1), (8, 768, 64, 128, 0), (8, 512, 200, 128, 0), (8, 384, 200, 96, 0),
        (8, 256, 200, 128, 1), (8, 128, 300, 96, 1), (1, 768, 300, 384, 0), (2, 768, 128, 200, 1), (2, 640, 33, 1000, 1), (8, 768, 33, 384, 0),
        (1, 640, 300, 20, 1), (8, 768, 16, 4096, 1), (8, 496, 1, 32768, 0), (8, 896, 1, 32768, 0),
        (8, 256, 64, 97, 0), (8, 256, 128, 128, 0), (8, 256, 63, 128, 1), (8, 256, 129, 128, 1), (8, 256, 128, 96, 1), (8, 256, 128, 129, 1),
        (8, 128, 128, 128, 0), (8, 128, 120, 128, 0), (8, 128, 119, 128, 1)]
    shapes = [dict(H_kv=h, H_q=h, r_k=r, L=L, batch=b) for h, r, b, L, _ in line]
    for case, p in zip(line, plan_of(shapes)):
        assert p["factor_kept"] == case[4], case
    cases = [dict(H_kv=h, H_q=h, r_k=r, L=L, batch=b) for h, b, L in tiles.KEPT for r in tiles.KEPT_RANKS]
    assert all(p["factor_kept"] for p in plan_of(cases))
    # nothing is divided by zero or wraps around at the ends of what the call takes
    plan_of([dict(H_kv=h, H_q=h, r_k=512, L=L, batch=b) for h, b in ((1, 1), (1, 65535), (255, 257)) for L in (1, 1 << 24)])

"""GPU parity of NHWC convolutions of few channels whose image rows are held in LDS (run_tile_rows) at the sizes where the rows, the runs and their
last pieces can go wrong, and of what a piece must not bring in from beyond its run.  Held to the oracle, and bit for bit over relaunch, order
and per-die lists (run_all_modes)."""
import numpy as np
import pytest
import torch

import paper_1901_10008_amd as sk

import sk_harness as H
from test_gpu_parity import c, run_all_modes

pytestmark = pytest.mark.gpu

FORMS = {
    # stems on RGB: filters, strides, output rows shorter and longer than a block of 128, channels up to the limit and beyond it (patches)
    "stems": [c(hw, hw, 3, co, r, r, r // 2, r // 2, dt, st=st) for dt in ("bf16", "f16", "f32")
              for hw, co, r, st in ((24, 32, 3, 1), (25, 48, 5, 2), (33, 64, 7, 2), (57, 64, 7, 1), (140, 7, 3, 1), (41, 65, 3, 2))],
    # runs of one piece, one element more, one less than two; even and odd steps between patches; runs shorter than a piece (patches)
    "runs": [c(20, 21, ci, 40, 3, s, 1, s // 2, dt, st=st) for dt in ("bf16", "f32") for ci, s, st in
             ((1, 8, 1), (1, 9, 3), (3, 3, 1), (5, 3, 1), (4, 4, 1), (7, 5, 2), (9, 3, 1), (11, 1, 2), (13, 3, 3), (1, 3, 1), (15, 1, 1))],
    # padding on one side only, beyond the filter, and none; one row, one column, images no wider than a filter
    "padding": [c(13, 17, 3, 20, 5, 5, 0, 0), c(13, 17, 3, 20, 5, 5, 4, 1), c(12, 12, 3, 20, 3, 3, 5, 6, st=2), c(1, 200, 3, 16, 1, 3, 0, 1),
                c(200, 3, 3, 16, 3, 3, 1, 1), c(150, 5, 3, 33, 7, 7, 3, 3, "f16"), c(3, 100, 6, 64, 5, 5, 2, 2), c(129, 3, 5, 8, 3, 3, 1, 1, "f32")],
    # windows of five and six pieces a thread (all others here take one to four)
    "windows": [c(40, 260, 3, 16, 5, 5, 2, 2, st=3), c(40, 190, 9, 16, 3, 3, 1, 1, st=2), c(40, 130, 9, 24, 5, 5, 2, 2, "f16", st=2),
                c(40, 260, 3, 16, 5, 5, 2, 2, "f32"), c(40, 75, 7, 16, 3, 3, 1, 1, "f32", st=2)],
    # several images: blocks in one each, and blocks that would not be (patches)
    "images": [c(16, 8, 3, 24, 3, 3, 1, 1, nb=3), c(15, 15, 3, 64, 3, 3, 1, 1, nb=2), c(32, 16, 5, 30, 5, 5, 2, 2, st=2, nb=4, dtype="f16"), c(16, 16, 3, 24, 3, 3, 1, 1, "f32", nb=3)],
}


@pytest.mark.parametrize("off", [0, 2, 4])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_rows(name, off):
    specs = [s for s in FORMS[name] if off != 2 or s.dtype != "f32"]
    run_all_modes(specs, seed=61, label=f"{name} at {off}", a_off=off, b_off=off, c_off=off)


def test_the_stem_of_a_residual_network():
    """7x7 on 224x224x3, two of them in one plan of their type (in fp32 as patches: their window does not fit LDS)."""
    for dt in ("bf16", "f16", "f32"):
        run_all_modes([c(224, 224, 3, 64, 7, 7, 3, 3, dt, st=2)] * 2, seed=62, label=dt)


# Enough tiles of few-channel operators for runs of several blocks: last blocks of 8 to 126 pixels, blocks of several rows of the image and within one,
# images whose tiles are joined only within each, steps between patches that are even and odd, runs of one to four and six pieces.
RUNS = {
    "bf16": [c(220, 220, 3, 8, 7, 7, 3, 3, st=2), c(111, 111, 5, 12, 5, 5, 2, 2), c(140, 70, 5, 9, 3, 3, 1, 1, nb=2), c(10, 1203, 1, 16, 3, 8, 1, 4)] * 6,
    "f16": [c(113, 113, 1, 7, 5, 9, 2, 4, "f16"), c(128, 100, 3, 64, 3, 3, 1, 1, "f16"), c(200, 63, 9, 10, 5, 5, 2, 2, "f16"), c(225, 227, 3, 5, 7, 7, 0, 0, "f16", st=2)] * 6,
    "f32": [c(111, 111, 3, 8, 5, 5, 2, 2, "f32"), c(158, 80, 1, 12, 3, 4, 1, 2, "f32"), c(94, 129, 2, 33, 3, 3, 1, 1, "f32"), c(70, 91, 5, 6, 3, 3, 1, 1, "f32", nb=2)] * 6,
}


@pytest.mark.parametrize("dtype", sorted(RUNS))
def test_runs_of_several_blocks(dtype):
    """One record takes several blocks of 128 pixels, the next one's rows on their way while one is multiplied.  run_all_modes compares them with the oracle
    and bit for bit with plans that have lists, where nothing is joined."""
    specs = RUNS[dtype]
    b = H.Batch(specs, seed=64)
    with b.plan() as plan:
        records = H.device_records(plan)
        blocks = {p: max(-(-r[6] // 128) for r in records if r[0] == p) for p in range(len(specs))}
        assert all(n >= 2 for n in blocks.values()), blocks
        partial = {r[6] % 128 for r in records if r[6] > 128}
        assert len(partial) > 1, partial
    with b.plan(xcd_part=32) as plan:
        assert max(r[6] for r in H.device_records(plan)) <= 128
    del b
    run_all_modes(specs, seed=64, label=dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_pieces_bring_in_nothing_from_beyond_their_run(dtype):
    """Infinities in one column of an image stay with the outputs whose filters cover it: all others are as without them."""
    specs = [c(17, 31, 3, 40, 3, 3, 1, 1, dtype), c(40, 19, 3, 64, 5, 5, 2, 2, dtype, st=2), c(30, 30, 5, 16, 3, 3, 1, 1, dtype)]
    bits = []
    for spoilt in (False, True):
        b = H.Batch(specs, seed=63)
        if spoilt:
            for s, buf in zip(specs, b.bufs[::2]):
                buf.view(H._T_REAL[dtype])[:s.H * s.W * s.Cin].view(s.H, s.W, s.Cin)[:, 9] = float("inf")
        with b.plan() as plan:
            sk.sk_launch(plan, H.stream_handle())
            torch.cuda.synchronize()
        bits.append(b.all_output_bits())
    for s, clean, got in zip(specs, *bits):
        wo = (s.W + 2 * s.pad_w - s.S) // s.stride + 1
        first = np.arange(wo) * s.stride - s.pad_w
        far = (first > 9) | (first + s.S <= 9)
        clean, got = clean.reshape(-1, wo, s.Cout), got.reshape(-1, wo, s.Cout)
        assert far.any() and np.array_equal(clean[:, far], got[:, far]), s
        assert not np.array_equal(clean, got), s

"""GPU parity of the paths for operands at any address and for channel-major images at the sizes where their
addressing can go wrong: runs shorter than a 16-byte piece, reduction lengths one below to one above a multiple of
one, filters wider than the image or than 32 taps, planes of an odd number of pixels over several images.  Held to
the oracle like every other shape (gate and order-free rounding bound), and bit for bit over relaunch, order and
per-die lists (run_all_modes)."""
import numpy as np
import pytest
import torch

import paper_1901_10008_amd as sk

import sk_harness as H
from test_gpu_parity import c, g, nchw, run_all_modes

pytestmark = pytest.mark.gpu

CASES = {
    # weight-streaming classes, 1 to 64 rows: K from one piece to several chunks, every remainder; padded rows below
    "skinny_tails": [g(m, 70, k, dt) for dt in ("bf16", "f32") for m, k in
                     ((1, 9), (5, 15), (16, 71), (17, 129), (32, 130), (33, 251), (48, 516), (64, 1021), (7, 2051), (1, 4099))],
    # a reduction cut into slices (the last one ragged)
    "skinny_slices": [g(3, 64, 9001), g(20, 33, 5003, "f16"), g(60, 40, 3001, "f32")],
    # fewer elements than a piece in a row, and fewer than a piece in the whole operand
    "short_rows": [g(1, 3, 2), g(300, 90, 5), g(200, 130, 3, "f32"), g(2, 500, 7), g(1, 700, 6, "f16")],
    # blocks of 128 x 128: K around multiples of a piece and of a stage
    "blocks": [g(130, 129, k, dt) for dt in ("bf16", "f16", "f32") for k in (33, 63, 65, 127, 193)],
    # image runs: 1x1 with few channels, 3x3 on RGB, odd channel counts, an image narrower than the filter
    "runs": [c(20, 20, 3, 40, 1, 1, 0, 0), c(24, 22, 3, 64, 3, 3, 1, 1, st=2), c(21, 23, 7, 33, 3, 3, 1, 1, "f32"),
             c(19, 3, 9, 70, 5, 5, 2, 2), c(30, 30, 1, 20, 7, 7, 3, 3, "f16"), c(15, 17, 13, 130, 3, 3, 0, 0, nb=3),
             c(40, 2, 3, 16, 3, 3, 1, 3), c(12, 12, 100, 24, 1, 1, 1, 1, st=2), c(9, 14, 12, 72, 1, 7, 0, 3)],
    # channel-major: filters of more than 32 columns, odd planes over several images, pad beyond the filter, stages
    # that end inside a channel
    "planes": [nchw(6, 60, 3, 40, 1, 41, 0, 20), nchw(45, 7, 2, 24, 33, 2, 4, 1, "f16"), nchw(7, 7, 33, 70, 1, 1, 0, 0, nb=5),
               nchw(9, 11, 20, 130, 3, 3, 1, 1, "f32", nb=3), nchw(13, 13, 17, 64, 2, 2, 2, 2), nchw(30, 30, 8, 12, 5, 5, 2, 2, st=3),
               nchw(14, 14, 96, 200, 1, 1, 0, 0, "f16")],
    # channel-major, filters that overhang a small image: the scalar offset of the last taps lies beyond the image
    "overhang": [nchw(1, 1, 64, 70, 3, 3, 1, 1), nchw(2, 2, 32, 40, 5, 5, 2, 2, nb=30), nchw(3, 3, 32, 70, 7, 7, 3, 3, "f16"),
                 nchw(1, 64, 8, 40, 5, 1, 2, 0), nchw(70, 1, 8, 33, 1, 5, 0, 2, "f32"), nchw(1, 1, 24, 30, 3, 3, 1, 1, "f32", nb=129)],
    # channel-major, image size kept (pixels in a row under every tap): planes smaller than a piece and a block, planes and channel
    # counts around multiples of a piece, several images that whole pieces fit into and that they do not
    "kept_sizes": [nchw(3, 3, 40, 70, 3, 3, 1, 1), nchw(8, 8, 24, 130, 3, 3, 1, 1, nb=3), nchw(7, 9, 33, 40, 3, 3, 1, 1, nb=2),
                   nchw(1, 17, 19, 20, 1, 3, 0, 1, "f16"), nchw(23, 1, 9, 65, 3, 1, 1, 0), nchw(12, 10, 65, 64, 1, 1, 0, 0, nb=2),
                   nchw(11, 13, 7, 129, 3, 3, 1, 1, "f32"), nchw(6, 6, 50, 30, 3, 3, 1, 1, "f32", nb=4), nchw(29, 31, 16, 16, 1, 1, 0, 0, "f32")],
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_any_alignment_edges(name):
    run_all_modes(CASES[name], seed=41, label=name)


@pytest.mark.parametrize("name", ["skinny_tails", "blocks", "runs", "planes", "overhang", "kept_sizes"])
def test_any_alignment_edges_at_odd_addresses(name):
    """The same at addresses that are aligned to an element only, GEMMs in rows padded by an odd number of elements."""
    off = 4  # bytes: whole elements of every type, no multiple of a piece
    pads = {} if name in ("runs", "planes", "overhang", "kept_sizes") else {"pad_lda": 5, "pad_ldb": 3, "pad_ldc": 1}
    run_all_modes(CASES[name], seed=42, label=name + " at odd addresses", a_off=off, b_off=off, c_off=off, **pads)


def test_padding_whose_width_in_elements_does_not_fit_32_bits():
    """One pixel of 8193 channels in the middle of 262144 columns of padding on either side, sampled every 1024 columns."""
    run_all_modes([c(1, 1, 8193, 3, 1, 1, 0, 1 << 18, st=1024), c(1, 1, 8193, 70, 1, 1, 0, 1 << 18, "f16", st=1024),
                   nchw(1, 1, 8193, 3, 1, 1, 0, 1 << 18, st=1024), c(1, 1, 8200, 66, 1, 1, 0, 1 << 18, st=1024)], seed=43, label="wide padding")


def test_cut_records_without_device_memory():
    """Records that are cut (one long odd operator per type) run the same through sk_launch_static, which plans for a device it
    does not know yet."""
    b = H.Batch([g(300, 130, 1001), g(200, 200, 501, "f16"), g(300, 130, 501, "f32"), c(20, 20, 33, 130, 3, 3, 1, 1)], seed=44)
    with b.plan() as plan:
        assert sk.sk_plan_grid(plan) > sk.sk_plan_num_tiles(plan)  # more workgroups than records in the table: some are cut
        sk.sk_launch(plan, H.stream_handle())
        torch.cuda.synchronize()
        H.check_against_oracle(b, "cut records")
        bits = b.all_output_bits()
    with b.plan(host_only=1) as plan:
        b.reset_outputs()
        sk.sk_launch_static(plan, H.stream_handle())
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(bits, b.all_output_bits())):
            assert np.array_equal(x, y), f"operator {i} differs through the static scratch"

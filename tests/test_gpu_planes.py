"""GPU parity of channel-major convolutions whose pixels are read in 16-byte pieces (run_tile_planes) at the sizes where the pieces, the
bits of the pixels to keep and the LDS images can go wrong, of the forms beside them that keep the single-element path, and of what a tap
outside the image must not bring in.  Held to the oracle, and bit for bit over relaunch, order and per-die lists (run_all_modes)."""
import numpy as np
import pytest
import torch

import paper_1901_10008_amd as sk

import sk_harness as H
from test_gpu_parity import nchw, run_all_modes

pytestmark = pytest.mark.gpu

FORMS = {
    # planes of one pixel less and more than a piece, a block of 64 and of 128, in rows of one pixel and one row of them
    "plane_sizes": [nchw(h, w, 16, 40, r, s, r // 2, s // 2, dt) for dt in ("f16", "f32")
                    for h, w, r, s in ((1, 7, 1, 3), (1, 8, 1, 3), (9, 1, 3, 1), (1, 9, 3, 3), (63, 1, 1, 1), (8, 8, 3, 3), (5, 13, 3, 3), (127, 1, 3, 3),
                                       (1, 129, 3, 3), (16, 8, 1, 1), (43, 3, 3, 3))],
    # filter rows: one to four, with less and more padding than keeps the height (five: single elements)
    "filter_rows": [nchw(12, 10, 24, 70, r, 3, p, 1) for r, p in ((1, 0), (2, 0), (2, 1), (2, 2), (3, 0), (3, 2), (4, 0), (4, 1), (4, 3), (5, 2))],
    # channels: stages that end inside a channel, before and behind a whole piece of the weight rows
    "channels": [nchw(10, 12, ci, co, 3, 3, 1, 1, dt) for dt in ("bf16", "f32") for ci, co in ((1, 64), (5, 65), (7, 63), (8, 128), (9, 129), (57, 200))],
    # several images: pieces that lie in one each, and pieces that would not (single elements)
    "images": [nchw(h, w, 24, 72, 3, 3, 1, 1, dt, nb=n) for dt in ("f16", "f32") for h, w, n in ((4, 4, 9), (7, 7, 3), (14, 14, 2), (2, 6, 20), (5, 5, 6))],
    # few output pixels against many channels (reduction slices), and a wide rectangle of a weight-streaming class
    "slices": [nchw(7, 7, 512, 200, 3, 3, 1, 1), nchw(7, 7, 200, 2048, 1, 1, 0, 0, "f16"), nchw(14, 14, 256, 130, 3, 3, 1, 1, "f32")],
}


@pytest.mark.parametrize("off", [0, 2, 4])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_planes(name, off):
    specs = [s for s in FORMS[name] if off != 2 or s.dtype != "f32"]
    run_all_modes(specs, seed=51, label=f"{name} at {off}", a_off=off, b_off=off, c_off=off)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_taps_outside_the_image_bring_nothing_in(dtype):
    """Infinities in the last column, row, and channel of an image stay with the outputs whose taps name them: all others are as
    without them."""
    specs = [nchw(9, 11, 12, 40, 3, 3, 1, 1, dtype, nb=2), nchw(8, 8, 12, 70, 3, 3, 1, 1, dtype, nb=2), nchw(13, 7, 9, 40, 1, 1, 0, 0, dtype)]
    bits = []
    for spoilt in (False, True):
        b = H.Batch(specs, seed=52)
        if spoilt:
            for s, buf in zip(specs, b.bufs[::2]):
                real = buf.view(H._T_REAL[dtype])[:s.Nb * s.Cin * s.H * s.W].view(s.Nb, s.Cin, s.H, s.W)
                real[0, -1, :, -1] = float("inf")
                real[0, -1, -1, :] = float("inf")
        with b.plan() as plan:
            sk.sk_launch(plan, H.stream_handle())
            torch.cuda.synchronize()
        bits.append(b.all_output_bits())
    for s, clean, got in zip(specs, *bits):
        shape = (s.Nb, s.Cout, s.H, s.W)
        clean, got = clean.reshape(shape), got.reshape(shape)
        p = s.R // 2
        far = np.ones((s.H, s.W), bool)
        far[s.H - 1 - p:, :] = False
        far[:, s.W - 1 - p:] = False
        assert np.array_equal(clean[0][:, far], got[0][:, far]), s
        assert np.array_equal(clean[1:], got[1:]), s
        assert not np.array_equal(clean[0], got[0]), s

"""GPU parity of size-keeping 3x3 convolutions of 64 channels run with their weights in registers: image
widths from three pixels to the widest its ring takes, images that end inside a block, several images, fewer channels out than a
wave makes, records of one to many blocks; held to the oracle, bit for bit to the tile kernels (same order of summation) and to a
relaunch; and beside operators of other kinds."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_1901_10008_amd as sk

import sk_harness as H
from test_gpu_parity import c, g

pytestmark = pytest.mark.gpu

CASES = {
    # the last pixels of a block, a record, an image: 128 +- 1, 256 +- 1 outputs, and 56 x 56
    "edges": [c(127, 1, 64, 64, 3, 3, 1, 1), c(43, 3, 64, 64, 3, 3, 1, 1), c(64, 2, 64, 64, 3, 3, 1, 1), c(51, 5, 64, 64, 3, 3, 1, 1),
              c(16, 16, 64, 64, 3, 3, 1, 1), c(1, 63, 64, 64, 3, 3, 1, 1, nb=3), c(56, 56, 64, 64, 3, 3, 1, 1)],
    # the widest image of the ring; several images in a block, and one over blocks
    "images": [c(9, 63, 64, 64, 3, 3, 1, 1), c(3, 3, 64, 64, 3, 3, 1, 1, nb=31), c(1, 1, 64, 64, 3, 3, 1, 1, nb=300), c(23, 23, 64, 64, 3, 3, 1, 1, nb=2)],
    # channels out
    "channels": [c(20, 20, 64, n, 3, 3, 1, 1) for n in (8, 24, 32, 40, 56, 64)],
}


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_window_plans(name, dtype):
    specs = [dataclasses.replace(s, dtype=dtype) for s in CASES[name]]
    b = H.Batch(specs, seed=61)

    def launch(plan, call=sk.sk_launch):
        b.reset_outputs()
        call(plan, H.stream_handle())
        torch.cuda.synchronize()
        return b.all_output_bits()

    with b.plan() as plan:  # fewer tiles than workgroups: the tile kernels
        assert sk.sk_plan_num_tiles(plan) < 500 and not H.runs_of_pixels(plan)
        tiles = launch(plan)
        H.check_against_oracle(b, f"tiles {name}")
        n = sk.sk_plan_num_tiles(plan)
    for prm in ({"grid_limit": 1}, {"grid_limit": 3}, {"grid_limit": n - 1}, {"grid_limit": 7, "stamps": 1}):
        with b.plan(**prm) as plan:
            assert sk.sk_plan_grid(plan) <= prm["grid_limit"]
            assert H.runs_of_pixels(plan) == list(range(len(specs)))
            first = launch(plan)
            H.check_against_oracle(b, f"window {name} {prm}")
            again = launch(plan)
            for i, (x, y, z) in enumerate(zip(tiles, first, again)):
                assert np.array_equal(x, y) and np.array_equal(y, z), f"{name} {prm}: operator {i}"
            if "stamps" in prm:
                done, start, rate = sk.sk_plan_get_stamps(plan)
                assert rate > 0 and all(d > start for d in done)
    with b.plan(grid_limit=3, host_only=1) as plan:
        assert H.runs_of_pixels(plan) == list(range(len(specs)))
        for x, y in zip(tiles, launch(plan, sk.sk_launch_static)):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_outputs_past_the_caches(dtype):
    """Runs of pixels, tiles and blocks for any alignment beside an operator that makes the plan large: their outputs then leave past the
    caches, with the bits they have in a plan whose outputs do not."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float16
    weights, x, y = torch.zeros(90000 * 1024, dtype=t, device="cuda"), torch.ones(1024, dtype=t, device="cuda"), torch.empty(90000, dtype=t, device="cuda")
    large = sk.make_problem(g(1, 90000, 1024, dtype), x.data_ptr(), weights.data_ptr(), y.data_ptr())
    nchw = c(14, 14, 64, 60, 3, 3, 1, 1)
    nchw = dataclasses.replace(nchw, op="conv_nchw")
    for specs in (CASES["edges"][:5], [g(130, 200, 256), g(200, 64, 136), c(12, 12, 64, 130, 3, 3, 1, 1)],
                  [g(130, 129, 131), nchw, c(20, 20, 3, 64, 7, 7, 3, 3, st=2), g(70, 64, 128)]):
        b = H.Batch([dataclasses.replace(s, dtype=dtype) for s in specs], seed=63)
        bits = []
        for problems in (b.problems, b.problems + [large]):
            with sk.sk_plan_create(problems, sk.sk_plan_params_default(grid_limit=3, tail_div=0)) as plan:
                assert bool(H.runs_of_pixels(plan)) == (specs[0].Cin == 64)
                b.reset_outputs()
                sk.sk_launch(plan, H.stream_handle())
                torch.cuda.synchronize()
                H.check_against_oracle(b, f"{len(problems)} operators")
                bits.append(b.all_output_bits())
        for i, (p, q) in enumerate(zip(*bits)):
            assert np.array_equal(p, q), i


@pytest.mark.parametrize("other", [g(70, 64, 128), c(14, 14, 128, 64, 3, 3, 1, 1), c(14, 14, 64, 64, 3, 3, 1, 1, st=2), c(14, 14, 64, 64, 3, 3, 0, 0),
                                   c(14, 14, 64, 60, 3, 3, 1, 1), c(3, 64, 64, 64, 3, 3, 1, 1), c(14, 14, 64, 64, 3, 3, 1, 1, "f16")],
                         ids=["gemm", "channels", "stride", "padding", "columns", "width", "types"])
def test_plans_with_other_operators(other):
    """An operator that keeps its tiles beside runs of pixels (another element type: no runs at all)."""
    b = H.Batch(CASES["edges"][:5] + [other], seed=62)
    with b.plan(grid_limit=3) as plan:
        assert H.runs_of_pixels(plan) == ([] if other.dtype == "f16" else list(range(5)))
        b.reset_outputs()
        sk.sk_launch(plan, H.stream_handle())
        torch.cuda.synchronize()
        H.check_against_oracle(b, "window and another")

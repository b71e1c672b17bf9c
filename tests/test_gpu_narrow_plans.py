"""GPU parity of the kernel for plans of 128x64 LDS tiles alone (three workgroups per CU, two stage images): one to many
stages, rows and columns that end inside a tile, reduction tails, split reductions, every element type, the per-die
lists; and that an operator which does not fit such a plan takes the whole plan to the general kernel."""
import pytest
import torch

import paper_1901_10008_amd as sk
from oracle import planner as P

import sk_harness as H
from test_gpu_parity import c, g, run_all_modes

pytestmark = pytest.mark.gpu

SHAPES = {
    "bf16": [c(56, 56, 64, 64, 3, 3, 1, 1), c(12, 12, 128, 40, 3, 3, 1, 1, nb=2), c(31, 9, 64, 8, 5, 5, 2, 2, st=2), g(65, 64, 64), g(300, 33, 72),
             g(129, 64, 8), g(200, 5, 1096), c(9, 9, 64, 64, 1, 1, 0, 0, nb=3)],
    "f16": [g(130, 64, 4096, "f16"), c(14, 14, 256, 64, 3, 3, 1, 1, "f16"), g(70, 17, 136, "f16")],
    "f32": [c(10, 10, 32, 48, 3, 3, 1, 1, "f32", nb=2), g(131, 50, 104, "f32"), g(140, 64, 36, "f32")],
}


@pytest.mark.parametrize("dtype", sorted(SHAPES))
def test_narrow_plans(dtype):
    run_all_modes(SHAPES[dtype], seed=51, label="narrow " + dtype)
    b = H.Batch(SHAPES[dtype], seed=52)
    for prm in ({"tile_bytes_min": 16384, "tile_bytes_max": 16384}, {"grid_limit": 5}, {"xcd_part": 2, "grid_limit": 37}):
        with b.plan(**prm) as plan:
            assert {t["cls"] for t in P.decode(sk.sk_plan_get_tiles(plan))} == {P.CLS_TILE_128x64}
            for _ in range(2):
                b.reset_outputs()
                sk.sk_launch(plan, H.stream_handle())
                torch.cuda.synchronize()
                H.check_against_oracle(b, f"narrow {dtype} {prm}")


@pytest.mark.parametrize("other", [g(70, 40, 1001), c(14, 14, 24, 64, 3, 3, 1, 1), c(14, 14, 64, 64, 7, 7, 3, 3), g(100, 64, 128, "f16"), g(8, 64, 64)],
                         ids=["odd", "channels", "taps", "types", "skinny"])
def test_plans_that_are_not_narrow(other):
    run_all_modes(SHAPES["bf16"][:2] + [other], seed=53, label="narrow and another")

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


def short_tiles(dtype, tiles):
    """One-stage 128x64 tiles: GEMMs of up to 1280 rows, a row short of the last tile."""
    rows, out = 128 * tiles - 1, []
    while rows > 0:
        out.append(g(max(65, min(1280, rows)), 40, 32, dtype))
        rows -= 1280
    return out


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("per_cu,workgroups", [(0.5, None), (1.5, None), (2.25, 3), (2.75, 2), (16, 3)])
def test_narrow_kernel_where_it_pays(dtype, per_cu, workgroups):
    """The numbers of tiles at which the rule changes sides, seen in the grid: three workgroups per compute unit or two."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    b = H.Batch(short_tiles(dtype, int(per_cu * cus)), seed=54)
    with b.plan() as plan:
        n = sk.sk_plan_num_tiles(plan)
        assert n == int(per_cu * cus)
        assert sk.sk_plan_grid(plan) == (n if workgroups is None else min(n, workgroups * cus))
        sk.sk_launch(plan, H.stream_handle())
        torch.cuda.synchronize()
        H.check_against_oracle(b, f"{n} tiles of {dtype}")


@pytest.mark.parametrize("other", [g(70, 40, 1001), c(14, 14, 24, 64, 3, 3, 1, 1), c(14, 14, 64, 64, 7, 7, 3, 3), g(100, 64, 128, "f16"), g(8, 64, 64)],
                         ids=["odd", "channels", "taps", "types", "skinny"])
def test_plans_that_are_not_narrow(other):
    run_all_modes(SHAPES["bf16"][:2] + [other], seed=53, label="narrow and another")
    # in the numbers at which a narrow plan gets three workgroups per compute unit it gets two
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    b = H.Batch(short_tiles("bf16", int(2.25 * cus)) + [other], seed=55)
    with b.plan() as plan:
        assert sk.sk_plan_num_tiles(plan) > 2 * cus and sk.sk_plan_grid(plan) == 2 * cus

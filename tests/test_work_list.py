"""The device's work list (long records cut, operators of one deadline the longest first): what it must cover, on the CPU under
the sanitizers, and results of records that only the list cuts, on the GPU."""
import ctypes
import os
import shutil

import pytest

import paper_1901_10008_amd as sk
import sk_harness as H
from workloads import Problem

from test_sanitizers import ENV, ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_work_list_under_sanitizers(tmp_path):
    exe = str(tmp_path / "work_list_driver")
    _run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"),
          "-I", os.path.join(ROOT, "paper_1901_10008_amd", "csrc"),
          os.path.join(ROOT, "tests", "sanitize", "work_list_driver.cpp"),
          os.path.join(ROOT, "paper_1901_10008_amd", "csrc", "planner.cpp"), "-o", exe])
    assert "work_list_driver: ok" in _run([exe], env=ENV)


def _slices(plan):
    """{operator: the reduction ranges of its outputs} of what the device runs, and the number of records."""
    records, got = H.device_records(plan), {}
    for r in records:
        got.setdefault(r[0], set()).add((r[8], r[9]))
    return got, len(records)


# Sixteen fp32 products whose list needs more than the 32 MiB that a table may have: two slices each for a chip of 512 workgroups.
BEYOND = [Problem(op="gemm", dtype="f32", M=128, N=2048, K=1024)] * 16


def test_slices_do_not_depend_on_the_grid_or_the_scratch():
    problems = [sk.make_problem(s, (1 << 40) + (i << 32), (1 << 40) + (i << 32) + (1 << 30), (1 << 40) + (i << 32) + (2 << 30))
                for i, s in enumerate(BEYOND)]
    for grid in (0, 3, 64, 256, 511, 513, 2000):
        with sk.sk_plan_create(problems, sk.sk_plan_params_default(host_only=1, grid_limit=grid)) as plan:
            got, n = _slices(plan)
            assert n == 2 * sk.sk_plan_num_tiles(plan)
            assert got == {i: {(0, 512), (512, 512)} for i in range(16)}, grid


def test_baseline_grid_of_plans_with_runs_of_pixels():
    """The one-launch-per-operator baseline of such a plan launches tiles: where the kernel of which three workgroups share a compute unit
    runs them, on three per compute unit, as in a plan of tiles."""
    L = sk.lib()
    L.sk_diag_plan_shape.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32]
    conv = Problem(op="conv", dtype="bf16", Nb=1, H=56, W=56, Cin=64, Cout=64, R=3, S=3, pad_h=1, pad_w=1)
    problems = [sk.make_problem(conv, (1 << 40) + (i << 32), (1 << 40) + (i << 32) + (1 << 30), (1 << 40) + (i << 32) + (2 << 30))
                for i in range(64)]
    with sk.sk_plan_create(problems[:20], sk.sk_plan_params_default(host_only=1)) as tiles, \
            sk.sk_plan_create(problems, sk.sk_plan_params_default(host_only=1)) as runs, \
            sk.sk_plan_create(problems, sk.sk_plan_params_default(host_only=1, grid_limit=600)) as limited:
        assert _slices(tiles)[1] == 500 and _slices(runs)[1] < sk.sk_plan_num_tiles(runs) == 1600
        for n in (1, 100, 400, 600, 640, 5000):
            assert L.sk_diag_plan_shape(runs.handle, n, 0) == L.sk_diag_plan_shape(tiles.handle, n, 0)
            assert 0 < L.sk_diag_plan_shape(runs.handle, n, 1) <= 512
            assert abs(L.sk_diag_plan_shape(limited.handle, n, 0)) == min(n, 600)
        assert L.sk_diag_plan_shape(runs.handle, 600, 0) == -600 and L.sk_diag_plan_shape(runs.handle, 5000, 0) == -768


# Few operators with long reductions: the launch would wait for single records, so the list slices them (LDS tiles from 32 stages
# on, blocks of any alignment from 12), and cuts wide weight-streaming records by columns.
def _cases():
    from test_gpu_parity import c, g, nchw
    return {
        "lds_tiles": [g(130, 129, 8192), g(70, 64, 4160, "f16"), g(200, 200, 4096, "f32"), c(9, 9, 256, 192, 3, 3, 1, 1), g(3, 64, 64)],
        "any_blocks": [g(130, 129, 3001), g(70, 33, 2049, "f16"), g(129, 65, 1501, "f32"), nchw(14, 14, 256, 130, 3, 3, 1, 1),
                       c(12, 12, 131, 70, 3, 3, 1, 1, "f32"), nchw(7, 7, 300, 200, 3, 3, 1, 1, "f16", nb=2)],
        "wide_streams": [g(1, 9000, 256), g(33, 5000, 260, "f32"), g(5, 4100, 516, "f16"), g(64, 3000, 128)] * 3,
    }


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["lds_tiles", "any_blocks", "wide_streams"])
def test_records_that_only_the_list_cuts(name):
    from test_gpu_parity import run_all_modes
    run_all_modes(_cases()[name], seed=51, label=name)

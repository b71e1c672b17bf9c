"""The device's work list (long records cut, operators of one deadline the longest first): what it must cover, on the CPU under
the sanitizers, and results of records that only the list cuts, on the GPU."""
import os
import shutil

import pytest

from test_sanitizers import ENV, ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_work_list_under_sanitizers(tmp_path):
    exe = str(tmp_path / "work_list_driver")
    _run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"),
          "-I", os.path.join(ROOT, "paper_1901_10008_amd", "csrc"),
          os.path.join(ROOT, "tests", "sanitize", "work_list_driver.cpp"),
          os.path.join(ROOT, "paper_1901_10008_amd", "csrc", "planner.cpp"), "-o", exe])
    assert "work_list_driver: ok" in _run([exe], env=ENV)


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

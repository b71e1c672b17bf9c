"""The device's records of few-channel convolutions (runs of tiles): on the CPU, that they cover every output once, that tiles are joined where that
pays and nowhere else, that plans with per-die lists keep the same slices, and that no cost of such a tile makes the planner slice it."""
import dataclasses
import os
import random
import shutil
import struct
import subprocess

import pytest

import paper_1901_10008_amd as sk
import sk_harness as H
from workloads import Problem


def _conv(hw, cin, cout, r, pad, stride=2, dtype="bf16", nb=1):
    return Problem(op="conv", dtype=dtype, Nb=nb, H=hw, W=hw, Cin=cin, Cout=cout, R=r, S=r, pad_h=pad, pad_w=pad, stride=stride)


LAYERS = [_conv(224, 3, 64, 7, 3), _conv(56, 128, 128, 3, 1), _conv(28, 256, 256, 3, 1), _conv(28, 512, 1024, 1, 0), _conv(14, 512, 512, 3, 1)]


def _records(specs, **prm):
    """The device's records, how many slices the table gives every operator, and its tiles."""
    at = 1 << 40
    problems = [sk.make_problem(s, at + (i << 32), at + (i << 32) + (1 << 30), at + (i << 32) + (2 << 30)) for i, s in enumerate(specs)]
    with sk.sk_plan_create(problems, sk.sk_plan_params_default(host_only=1, **prm)) as plan:
        table = struct.iter_unpack("<IHBBIIHHIII", sk.sk_plan_get_tiles(plan))
        return H.device_records(plan), {t[0]: t[3] for t in table}, sk.sk_plan_num_tiles(plan)


@pytest.mark.parametrize("specs,joined", [
    (LAYERS * 16, True),
    ([_conv(224, 3, 64, 7, 3, nb=2)] * 8 + LAYERS * 4, True),                        # (images of whole tiles)
    ([_conv(220, 3, 64, 7, 3, nb=3)] * 6 + LAYERS * 4, True),                        # (tiles of two images stay single)
    (LAYERS * 2, False),                                                             # too few tiles
    (LAYERS[:1] * 8 + LAYERS[1:] * 40, False),                                       # not a fifth of the work
    (LAYERS * 12 + [_conv(28, 512, 1024, 1, 0, dtype="f16")], False),                # two types
], ids=["downsampling", "images", "across", "few", "share", "types"])
def test_runs_cover_every_output_once(specs, joined):
    records, _, tiles = _records(specs)
    assert any(r[6] > 128 for r in records) == joined
    rows = {}
    for p, cls, ks, S, m0, n0, m_len, n_len, k0, k_len, rect in records:
        if specs[p].Cin == 3:
            assert (ks, S, n0, n_len, k0, k_len) == (0, 1, 0, 64, 0, 147)
            rows.setdefault(p, []).append((m0, m0 + m_len))
    for p, s in enumerate(specs):
        if s.Cin == 3:
            hw = (s.H // 2) ** 2
            spans = sorted(rows[p])
            assert spans[0][0] == 0 and spans[-1][1] == s.Nb * hw and all(a[1] == b[0] for a, b in zip(spans, spans[1:]))
            across = [(a, b) for a, b in spans if a // hw != (b - 1) // hw]
            assert len(across) >= (s.Nb - 1 if hw % 128 else 0) and all(a % 64 == 0 and b - a <= 128 for a, b in across)
    assert (len(records) < tiles) == joined or not joined


def test_runs_of_operators_with_deadlines_are_short():
    """The first operators in the order of deadlines are not done with the launch's middle: an eighth of a workgroup's share of the launch at most, a third
    where nothing has a deadline or all have the same."""
    stem = _conv(224, 3, 64, 7, 3)
    deadlines = list(range(64, 0, -1))
    share = 64 * 98 * 9000 // 512 // 4500  # blocks
    longest = {}
    for name, at in (("none", [float("inf")] * 64), ("one", [2.0] * 64), ("own", deadlines)):
        records, _, _ = _records([dataclasses.replace(stem, deadline_ms=d) for d in at])
        longest[name] = max(r[6] for r in records) // 128
        order = [r[0] for r in records]
        assert order == sorted(order, key=lambda p: at[p])
    assert longest["none"] == longest["one"] == share // 3
    assert 1 < longest["own"] == share // 8


def _mix(seed):
    """Stems, whose tiles are joined, beside a few long reductions, which are sliced."""
    r = random.Random(seed)
    stems = [_conv(r.randint(150, 270), 3, 64, 7, 3, nb=r.choice([1, 1, 2])) for _ in range(r.randint(5, 24))]
    return stems + [_conv(r.randint(7, 26), r.randint(128, 2048), r.randint(128, 512), 3, 1, stride=1) for _ in range(r.randint(1, 6))]


@pytest.mark.parametrize("seed", [8, 46, 59, 72, 76])
def test_lists_and_grids_keep_the_slices(seed):
    """The reduction ranges of every 128 x 128 outputs, in a plan whose tiles are joined and some of whose rectangles only the list slices."""
    specs = _mix(seed)
    slices = []
    for prm in (dict(xcd_part=0), dict(xcd_part=32), dict(xcd_part=0, grid_limit=300)):
        records, table, _ = _records(specs, **prm)
        slices.append({(r[0], r[4] // 128 if specs[r[0]].Cin != 3 else 0, r[5] // 128, r[8], r[9]) for r in records})
        if not prm["xcd_part"]:
            assert any(r[6] > 128 for r in records)
            assert any(r[3] != table[r[0]] for r in records)
    assert slices[0] == slices[1] == slices[2]


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1901_10008_amd", "csrc")

# A plan of few stems beside many short tiles, where a long record would be sliced: none of the stems' is.
SLICES_CPP = r"""
#include <cstdio>
#include <limits>
#include <string>
#include "sk_internal.h"
int main() {
  std::vector<sk_problem> ps;
  for (int i = 0; i < 47; ++i) {
    const bool stem = i < 5;  // 64x64x3, 7x7, stride 2: eight tiles each; 56x56x64, 1x1: 25
    sk_problem p{};
    p.op = SK_CONV2D_NHWC, p.dtype = SK_BF16, p.Nb = 1, p.H = p.Wd = stem ? 64 : 56, p.Cin = stem ? 3 : 64, p.Cout = 64;
    p.R = p.S = stem ? 7 : 1, p.pad_h = p.pad_w = stem ? 3 : 0, p.stride = stem ? 2 : 1;
    p.deadline_ms = std::numeric_limits<double>::infinity();
    const uintptr_t at = ((uintptr_t)1 << 44) + ((uintptr_t)i << 32);
    p.A = (void *)at, p.B = (void *)(at + (1u << 30)), p.C = (void *)(at + (2ull << 30));
    ps.push_back(p);
  }
  sk_plan_params prm;
  sk_plan_params_default(&prm);
  prm.host_only = 1;
  sk::HostPlan hp;
  std::string err;
  if (sk::plan_host(ps.data(), (int32_t)ps.size(), &prm, hp, err) != SK_OK) return 1;
  if (!(hp.dev[0].flags & sk::FLAG_ROWS)) return 2;
  sk::WorkList w;
  for (const sk_tile &t : sk::device_list(hp, 512, false, w, true) ? w.work : hp.tiles)
    if (t.problem < 5 && t.S != 1) return 3;
  std::puts("slices: ok");
}
"""


# 64 stems: operators that run_tile_rows serves against ones of as many tiles that it does not (11x11: runs of five pieces): plan and list.
TIME_CPP = r"""
#include <chrono>
#include <cstdio>
#include <limits>
#include <string>
#include "sk_internal.h"
int main() {
  double best[2] = {1e9, 1e9};
  size_t records[2] = {0, 0};
  for (int rep = 0; rep < 60; ++rep)
    for (int other = 0; other < 2; ++other) {
      std::vector<sk_problem> ps;
      for (int i = 0; i < 64; ++i) {
        sk_problem p{};
        p.op = SK_CONV2D_NHWC, p.dtype = SK_BF16, p.Nb = 1, p.H = p.Wd = 224, p.Cin = 3, p.Cout = 64, p.stride = 2;
        p.R = p.S = other ? 11 : 7, p.pad_h = p.pad_w = other ? 5 : 3;
        p.deadline_ms = std::numeric_limits<double>::infinity();
        const uintptr_t at = ((uintptr_t)1 << 44) + ((uintptr_t)i << 32);
        p.A = (void *)at, p.B = (void *)(at + (1u << 30)), p.C = (void *)(at + (2ull << 30));
        ps.push_back(p);
      }
      sk_plan_params prm;
      sk_plan_params_default(&prm);
      prm.host_only = 1;
      sk::HostPlan hp;
      sk::WorkList w;
      std::string err;
      const auto from = std::chrono::steady_clock::now();
      if (sk::plan_host(ps.data(), (int32_t)ps.size(), &prm, hp, err) != SK_OK) return 1;
      sk::device_list(hp, 512, false, w, true);
      const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - from).count();
      best[other] = us < best[other] ? us : best[other];
      records[other] = w.work.empty() ? hp.tiles.size() : w.work.size();
    }
  std::printf("%.1f %.1f %zu %zu\n", best[0], best[1], records[0], records[1]);
}
"""


def _compiled(tmp_path, main, planner, flags="-O1"):
    (tmp_path / "planner.cpp").write_text(planner)
    (tmp_path / "main.cpp").write_text(main)
    exe = str(tmp_path / "driver")
    res = subprocess.run(["g++", "-std=c++17", flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(tmp_path / "main.cpp"),
                          str(tmp_path / "planner.cpp"), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


def _planner():
    with open(os.path.join(CSRC, "planner.cpp")) as f:
        return f.read()


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_tiles_of_few_channels_are_never_sliced(tmp_path):
    """Whatever the planner takes such a tile's start to cost: here so much that it outlasts what other records are sliced from."""
    text = _planner()
    assert text.count("ROWS_START = 6000") == 1
    exe = _compiled(tmp_path, SLICES_CPP, text.replace("ROWS_START = 6000", "ROWS_START = 40000"))
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and "slices: ok" in res.stdout, (res.returncode, res.stderr)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_runs_cost_the_planner_little(tmp_path):
    """The shortest of 60 plans with runs takes no more than twice the shortest of 60 without (1.1 times as measured; with the operator's form worked out for
    every record it was 3.6)."""
    res = subprocess.run([_compiled(tmp_path, TIME_CPP, _planner(), "-O2")], capture_output=True, text=True)
    assert res.returncode == 0
    runs, tiles, n, m = res.stdout.split()
    assert int(n) < 1000 < int(m)
    assert float(runs) < 2 * float(tiles), res.stdout

"""Build libsuperkernel.so (HIP, gfx950 only) in-tree next to this file."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsuperkernel.so")
CEILINGS_LIB = os.path.join(HERE, "libsk_ceilings.so")  # measuring aid of bench.py, not part of the ABI
SOURCES = ["superkernel.hip", "planner.cpp", "queue.cpp", "instances.hip", "scratch.hip"]
UNITS = 7  # units of compilation of instances.hip
HEADERS = ["kernels.hip.h", "sk_internal.h", os.path.join(ROOT, "include", "superkernel.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    # The tile queue's atomic is issued by one thread and its answer is wanted several loop steps
    # later.  The compiler's wave-level atomic combining reads the answer back at once, which
    # makes the wave wait for every load in flight at that point.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
]


DIAG_LIB = os.path.join(HERE, "libsuperkernel_diag.so")  # -DSK_DIAG_CLOCKS: per-tile phase stamps (tile_phases.py)
DIAG_ALL_LIB = os.path.join(HERE, "libsuperkernel_diag_all.so")  # the same with every workgroup of a launch stamped


def build_diag(verbose: bool = False, all_workgroups: bool = False) -> str:
    """The library once more with -DSK_DIAG_CLOCKS, as libsuperkernel_diag.so (a measuring aid: every tile
    of the first 16 workgroups stamps the device clock at its phase boundaries), or, with `all_workgroups`, as
    libsuperkernel_diag_all.so (512 workgroups, their first 24 tiles).  Not built by build()."""
    if all_workgroups:
        return build(force=True, verbose=verbose, extra=("-DSK_DIAG_CLOCKS", "-DSK_DIAG_WGS_N=512", "-DSK_DIAG_TILES_N=24"),
                     lib=DIAG_ALL_LIB, ceilings=False, tag="diag_all")
    return build(force=True, verbose=verbose, extra=("-DSK_DIAG_CLOCKS",), lib=DIAG_LIB, ceilings=False, tag="diag")


def build(force: bool = True, verbose: bool = False, extra=(), lib: str = LIB, ceilings: bool = True, tag: str = "") -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    if not force and os.path.exists(lib):
        newest = max(os.path.getmtime(p) for p in srcs + [os.path.join(CSRC, h) if not os.path.isabs(h) else h
                                                          for h in HEADERS])
        if os.path.getmtime(lib) >= newest:
            return lib
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    o_hip = os.path.join(obj_dir, f"superkernel{tag}.o")
    o_cpp = os.path.join(obj_dir, "planner.o")
    o_queue = os.path.join(obj_dir, "queue.o")
    o_scratch = os.path.join(obj_dir, "scratch.o")
    # the kernels are compiled side by side (a diagnostic build, -DSK_DIAG_CLOCKS, compiles them with superkernel.hip)
    units = [] if "-DSK_DIAG_CLOCKS" in extra else list(range(UNITS))
    o_units = [os.path.join(obj_dir, f"instances{u}{tag}.o") for u in units]
    compiles = [[hipcc, *HIPCC_FLAGS, *extra, *inc, f"-DSK_UNIT={u}", "-c", srcs[3], "-o", o] for u, o in zip(units, o_units)] + [
        [hipcc, *HIPCC_FLAGS, *extra, *inc, "-c", srcs[0], "-o", o_hip],
        [hipcc, *HIPCC_FLAGS, *inc, "-c", srcs[4], "-o", o_scratch],
        ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", *inc, "-c", srcs[1], "-o", o_cpp],
        # host code that calls the HIP runtime (events): the host compiler with the runtime's headers
        ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", *inc, "-c", srcs[2],
         "-o", o_queue],
    ]
    if ceilings:
        compiles.append([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
                         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                         os.path.join(CSRC, "ceilings.hip"), "-o", CEILINGS_LIB])
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", o_hip, *o_units, o_cpp, o_queue, o_scratch, "-o", lib]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass warns that it does not know the packed-fp32 feature: harmless noise
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("build step failed: " + " ".join(cmd) + "\n" + err)
        if verbose and err.strip():
            print(err)

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        list(pool.map(run, compiles))
    run(link)
    return lib


if __name__ == "__main__":
    print(build(force=True, verbose=True))

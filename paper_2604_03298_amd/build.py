"""Builds libenec.so (HIP, gfx950) in-tree with hipcc.  `python -m paper_2604_03298_amd.build`.

libenec_test.so is the same library with ENEC_TEST_HOOKS defined for the host code: there the environment
variable ENEC_SPIN_LIMIT lowers the bound of the scan's waits, which the tests of that bound need.

The host code (csrc/enec_api.hip, csrc/enec_pipeline.hip), the compression kernels for one tuple per data block
(csrc/enec_per_block.hip, its fp32 kernels with deferred stores apart) and for tensors of one block (csrc/enec_single.hip), the
decompression kernels (csrc/enec_decompress.hip, those for one stream apart) and the eighteen tables of compression kernels
(csrc/enec_kernels.hip, once per element format, group length and kind of block size) are compiled side by side into
_build/*.o and linked into libenec.so.
"""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libenec.so")
TEST_LIB = os.path.join(HERE, "libenec_test.so")      # the same library with ENEC_TEST_HOOKS (tests of the bounded waits)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
SOURCES = [os.path.join(CSRC, "enec_api.hip"), os.path.join(CSRC, "enec_kernels.hip"),
           os.path.join(CSRC, "enec_per_block.hip"), os.path.join(CSRC, "enec_pipeline.hip"),
           os.path.join(CSRC, "enec_decompress.hip"), os.path.join(CSRC, "enec_single.hip")]
HEADERS = [os.path.join(CSRC, "enec_device.hpp"), os.path.join(CSRC, "enec_kernels.hpp"),
           os.path.join(CSRC, "enec_per_block.hpp"), os.path.join(CSRC, "enec_decompress.hpp"),
           os.path.join(CSRC, "enec_single.hpp"),
           os.path.join(ROOT, "include", "enec.h")]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=off",
         "-fPIC", "-I", os.path.join(ROOT, "include")]


def _units():
    units = [("enec_api.o", [SOURCES[0]]), ("enec_api_test.o", ["-DENEC_TEST_HOOKS", SOURCES[0]]),
             # (no constants kept in registers over a loop with sixteen packers: compress_per_block_stream_kernel in
             # enec_per_block.hpp, where both sides' figures stand: fp32 is faster with them; the unit's other kernel is the same either way)
             ("enec_per_block.o", ["-DENEC_FP32=0", "-mllvm", "-disable-machine-licm", SOURCES[2]]),
             ("enec_per_block_fp32.o", ["-DENEC_FP32=1", SOURCES[2]]),
             ("enec_pipeline.o", [SOURCES[3]]), ("enec_single.o", [SOURCES[5]]),
             ("enec_decompress.o", ["-DENEC_ONE=0", SOURCES[4]]), ("enec_decompress_one.o", ["-DENEC_ONE=1", SOURCES[4]])]
    for lpg in (2, 1, 4):           # lanes per group: group lengths 16, 8, 32
        for dt in (0, 2, 1):
            for logb in (14, 0):    # block size: the default one as a constant, any as an argument
                units.append((f"enec_kernels_dt{dt}_lpg{lpg}_b{logb}.o",
                              [f"-DENEC_DT={dt}", f"-DENEC_LPG={lpg}", f"-DENEC_LOGB={logb}", SOURCES[1]]))
    return units


def build(verbose: bool = False) -> str:
    """Compiles every HIP source for gfx950 (cross-compiles without a GPU) and returns the path."""
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(unit):
        name, args = unit
        cmd = ["hipcc"] + FLAGS + ["-c", "-o", os.path.join(OBJ, name)] + args
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
        return os.path.join(OBJ, name)

    workers = max(1, min(8, os.cpu_count() or 1))
    with ThreadPoolExecutor(workers) as pool:
        objects = list(pool.map(compile_one, _units()))
    api, api_test = os.path.join(OBJ, "enec_api.o"), os.path.join(OBJ, "enec_api_test.o")
    for lib, skip in ((LIB, api_test), (TEST_LIB, api)):
        cmd = ["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared", "-o", lib] + [o for o in objects if o != skip]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc (link) failed:\n" + res.stdout + res.stderr)
    return LIB


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS)


if __name__ == "__main__":
    print(build(verbose=True))

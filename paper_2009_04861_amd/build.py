"""Compiles the HIP library for gfx950 (hipcc cross-compiles without a GPU)."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(PKG, "csrc", "tm_kernels.hip")
TRAIN_PART = os.path.join(PKG, "csrc", "tm_train_part.hip")
LIB = os.path.join(PKG, "libtm_hip.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950",
    # packed fp32 instructions are not wanted on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the per-slot loops of the training kernel must unroll completely even for
    # 20 register slots, or the automata fall out of registers into scratch
    "-mllvm", "-pragma-unroll-threshold=1000000",
    "-fPIC",
]


TRAIN_PARTS = 8  # translation units that the forms of the training kernel are spread over


def build_library(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = "%s.tmp%d" % (LIB, os.getpid())
    units = [(SRC, [])] + [(TRAIN_PART, ["-DTM_TRAIN_PART=%d" % k]) for k in range(1, TRAIN_PARTS + 1)]
    objects = ["%s.%d.o" % (tmp, k) for k in range(len(units))]
    commands = [[hipcc] + HIPCC_FLAGS + defs + ["-c", src, "-o", obj] for (src, defs), obj in zip(units, objects)]
    commands.append([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objects + ["-o", tmp])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd, stderr=None if verbose else subprocess.DEVNULL)

    try:
        with ThreadPoolExecutor(min(len(units), os.cpu_count() or 1)) as pool:
            list(pool.map(run, commands[:-1]))
        run(commands[-1])
        os.replace(tmp, LIB)
    finally:
        for path in objects + [tmp]:
            if os.path.exists(path):
                os.remove(path)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))

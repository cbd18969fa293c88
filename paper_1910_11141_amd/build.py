"""Builds the HIP library (libnuts_hip.so) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libnuts_hip.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                      # a*b+c stays two roundings unless fma() is written out
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


# Kernels whose instances keep a chain's state in registers through a loop that is long and deep: hoisting constants and
# addresses out of it (the compiler's habit) fills the register file and spills the state itself (chip kernel: 400 bytes a
# lane; the others: nuts_gauss.hip).
NO_LICM = ["-mllvm", "-disable-machine-licm", "-mllvm", "-sink-insts-to-avoid-spills=1"]
# (pcvm.hip asks for the register limit of eight waves, not for eight waves, and names M0 among the registers that its assembly changes,
# which the compiler keeps for itself: it says so of every place)
EXTRA_FLAGS = {"nuts_chip.hip": NO_LICM, "nuts_gauss.hip": NO_LICM, "pcvm.hip": ["-Wno-pass-failed", "-Wno-inline-asm"]}


def flags_of(source):
    """The compiler flags of a translation unit."""
    return [f for f in FLAGS if f != "-shared"] + EXTRA_FLAGS.get(os.path.basename(source), [])


def sources():
    return [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]


def headers():
    inc = os.path.join(os.path.dirname(HERE), "include")
    return [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".h")] + \
           [os.path.join(inc, f) for f in sorted(os.listdir(inc))]


def is_stale() -> bool:
    if not os.path.exists(LIB_PATH):
        return True
    t = os.path.getmtime(LIB_PATH)
    return any(os.path.getmtime(p) > t for p in sources() + headers() + [os.path.abspath(__file__)])  # (the flags are here)


UBENCH_SRC = os.path.join(CSRC, "ubench", "issue_ubench.hip")
UBENCH_LIB = os.path.join(HERE, "libnuts_ubench.so")


def build(force: bool = True, verbose: bool = False) -> str:
    """The sampler library, and the instruction-issue microbenchmark as a library of its own."""
    if not force and not is_stale() and os.path.exists(UBENCH_LIB) and \
            os.path.getmtime(UBENCH_LIB) >= os.path.getmtime(UBENCH_SRC):
        return LIB_PATH
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in sources()]
        cmds = [[HIPCC] + flags_of(s) + ["-c", s, "-o", o] for s, o in zip(sources(), objects)]
        cmds.append([HIPCC] + FLAGS + [UBENCH_SRC, "-o", UBENCH_LIB])
        for cmd in cmds if verbose else []:
            print(" ".join(cmd), file=sys.stderr)
        with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as pool:  # one compiler per source
            list(pool.map(lambda cmd: subprocess.run(cmd, check=True), cmds))
        subprocess.run([HIPCC] + FLAGS + objects + ["-o", LIB_PATH], check=True)
    return LIB_PATH


if __name__ == "__main__":
    print(build(force=True, verbose=True))

"""Builds the HIP library (libnuts_hip.so) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import re
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


# The first of the registers in which the interpreter of small programs keeps its state without the compiler's knowledge (csrc/pcvm.hip).
PCVM_FIRST_REGISTER = 68


def faults_in_assembly(listing):
    """What is wrong in the assembly of a translation unit (its lines) that neither compiler nor assembler says.

    Lost reloads: a vector of registers that was spilled partly to accumulation registers and partly to scratch memory comes back, if it
    goes to accumulation registers, as copies from the highest register down and a load of the rest.  The load is marked as if it wrote the whole vector,
    and the copy before it is then deleted as dead: the register above the loaded ones keeps what was there (seen at a[116:119], of which a117 was
    written nowhere, in an instance of the element-wise kernel that is not built any more: wrong values throughout).  Only kernels that spill to
    both can have it.  Vectors here have two or four registers and begin at an even one; what is loaded are their first.  (A load of one even
    register could be of a value of 32 bits, too: then this says more than is the case.)

    Registers of the interpreter: see PCVM_FIRST_REGISTER."""
    faults, name, in_asm, block = [], None, False, []

    def look_at(block):
        for at, text in block:
            load = re.match(r"scratch_load_dword(x[234])? a(?:(\d+)|\[(\d+):(\d+)\]),.*Folded Reload", text)
            if not load:
                continue
            low, high = (int(load.group(2)),) * 2 if load.group(2) else (int(load.group(3)), int(load.group(4)))
            copied = [int(m.group(1)) for n, t in block if abs(n - at) <= 8 for m in [re.match(r"v_accvgpr_mov_b32 a(\d+),", t)] if m]
            if low % 2 == 0 and (high - low in (0, 2) or (high - low == 1 and high + 2 in copied)):
                faults.append(f"{name}: a reload may have lost a register: {text}")

    for at, line in enumerate(listing):
        text = line.strip()
        start = re.match(r"(_Z\w+):", text)
        if start:
            name, block = start.group(1), []
        if name is None:
            continue
        if re.match(r"\.LBB\w+:|\.Lfunc_end|s_c?branch|s_endpgm", text):
            look_at(block)
            block = []
        if text.startswith(".Lfunc_end"):
            name = None
            continue
        block.append((at, text))
        in_asm |= "ASMSTART" in text
        if not in_asm and "pcvm_small_kernel" in name and not text.startswith((".", ";")):
            code = text.split(";")[0]
            used = [int(r) for r in re.findall(r"\bv(\d+)\b", code)] + [int(r) for r in re.findall(r"\bv\[\d+:(\d+)\]", code)]
            if max(used, default=0) >= PCVM_FIRST_REGISTER:
                faults.append(f"{name}: the compiler uses a register of the interpreter's: {text}")
        in_asm &= "ASMEND" not in text
    return faults


UBENCH_SRC = os.path.join(CSRC, "ubench", "issue_ubench.hip")
UBENCH_LIB = os.path.join(HERE, "libnuts_ubench.so")


def build(force: bool = True, verbose: bool = False) -> str:
    """The sampler library, and the instruction-issue microbenchmark as a library of its own."""
    if not force and not is_stale() and os.path.exists(UBENCH_LIB) and \
            os.path.getmtime(UBENCH_LIB) >= os.path.getmtime(UBENCH_SRC):
        return LIB_PATH
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in sources()]
        cmds = [[HIPCC] + flags_of(s) + ["--save-temps=obj", "-c", s, "-o", o] for s, o in zip(sources(), objects)]
        cmds.append([HIPCC] + FLAGS + [UBENCH_SRC, "-o", UBENCH_LIB])
        for cmd in cmds if verbose else []:
            print(" ".join(cmd), file=sys.stderr)
        with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as pool:  # one compiler per source
            list(pool.map(lambda cmd: subprocess.run(cmd, check=True), cmds))
        for o in objects:
            with open(re.sub(r"\.hip\.o$", "-hip-amdgcn-amd-amdhsa-gfx950.s", o)) as listing:
                faults = faults_in_assembly(listing)
            if faults:
                raise RuntimeError("\n".join(faults))
        subprocess.run([HIPCC] + FLAGS + objects + ["-o", LIB_PATH], check=True)
    return LIB_PATH


if __name__ == "__main__":
    print(build(force=True, verbose=True))

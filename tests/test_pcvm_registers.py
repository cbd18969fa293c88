"""The virtual machine's step loop keeps its register files in registers that the compiler must not use (csrc/pcvm.hip):
the compiled kernels are read for any that it does."""
import os
import re
import subprocess

from paper_1910_11141_amd import build

FIRST_OF_THE_FILES = 68


def test_the_compiler_stays_below_the_register_files(tmp_path):
    src, out = os.path.join(build.CSRC, "pcvm.hip"), str(tmp_path / "pcvm.s")
    subprocess.run([build.HIPCC] + build.flags_of(src) + ["--offload-device-only", "-S", src, "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    kernels, name, in_asm = {}, None, False
    for line in open(out):
        start = re.match(r"(_Z\w*pcvm_small_kernel\w*):", line)
        if start:
            name = start.group(1)
            kernels[name] = -1
        if name is None or line.lstrip().startswith("."):
            continue
        in_asm |= "ASMSTART" in line
        if not in_asm:
            used = [int(r) for r in re.findall(r"\bv(\d+)\b", line)] + [int(r) for r in re.findall(r"\bv\[\d+:(\d+)\]", line)]
            kernels[name] = max([kernels[name]] + used)
        in_asm &= "ASMEND" not in line
        if "s_endpgm" in line:
            name = None
    assert len(kernels) == 6 and min(kernels.values()) > 0
    assert max(kernels.values()) < FIRST_OF_THE_FILES, kernels


def test_the_register_index_mode_is_declared(tmp_path):
    """s_set_gpr_idx_on writes M0: every piece of assembly that has it says so to the compiler."""
    src, out = os.path.join(build.CSRC, "pcvm.hip"), str(tmp_path / "pcvm.ll")
    subprocess.run([build.HIPCC] + build.flags_of(src) + ["--offload-device-only", "-S", "-emit-llvm", src, "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    pieces = [line for line in open(out) if "call" in line and "s_set_gpr_idx_on" in line]
    assert len(pieces) >= 6
    assert all("~{m0}" in line for line in pieces)

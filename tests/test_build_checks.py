"""What the build looks for in the compiled assembly (paper_1910_11141_amd/build.py)."""
import pytest

from paper_1910_11141_amd import build

HEAD = ["\t.text\n", "_ZN4nuts6kernelEv: ; @kernel\n", "; %bb.0:\n"]
TAIL = ["\ts_endpgm\n", ".Lfunc_end0:\n"]

# as compiled: a[116:119] out of a203, a254, a255 and scratch memory, the copy of a255 deleted
LOST = ["\tds_write_b128 v2, v[134:137] offset:48128\n", ".LBB0_191:                              ;   in Loop: Header=BB0_139 Depth=4\n",
        "\tv_accvgpr_mov_b32 a119, a203\n", "\tv_accvgpr_mov_b32 a118, a254\n", "\tscratch_load_dword a116, off, off       ; 4-byte Folded Reload\n",
        "\tv_mov_b64_e32 v[4:5], v[188:189]\n"]


@pytest.mark.parametrize("lines,found", [
    (LOST, 1),
    (["\tv_accvgpr_mov_b32 a11, a3\n", "\tscratch_load_dwordx2 a[8:9], off, off offset:16 ; 8-byte Folded Reload\n"], 1),   # a10 lost
    (["\tscratch_load_dwordx3 a[8:10], off, off offset:16 ; 12-byte Folded Reload\n"], 1),                                 # a11 lost
    (["\ts_endpgm\n", ".LBB0_2:\n"] + LOST, 1),                                                                              # beyond an early end
    (["\tscratch_load_dwordx4 a[116:119], off, off ; 16-byte Folded Reload\n"], 0),                                        # a whole vector
    (["\tv_accvgpr_mov_b32 a191, a65\n", "\tscratch_load_dwordx2 a[200:201], off, off ; 8-byte Folded Reload\n"], 0),
    (["\tv_accvgpr_mov_b32 a11, a3\n", "\ts_branch .LBB0_3\n", "\tscratch_load_dwordx2 a[8:9], off, off ; 8-byte Folded Reload\n"], 0),  # another block's
    (["\tv_accvgpr_mov_b32 a55, a63\n", "\tscratch_load_dword a63, off, off offset:556 ; 4-byte Folded Reload\n"], 0),      # 32 bits
    (["\tv_accvgpr_mov_b32 a119, a203\n", "\tscratch_load_dwordx2 v[116:117], off, off ; 8-byte Folded Reload\n"], 0),
])
def test_reloads_that_lost_a_register(lines, found):
    faults = build.faults_in_assembly(HEAD + lines + TAIL)
    assert len(faults) == found and all("_ZN4nuts6kernelEv" in f for f in faults)


def test_registers_of_the_interpreter():
    head = ["_ZN12_GLOBAL__N_117pcvm_small_kernelILb1ELb1ELb0EEEv6VmArgs9SmallArgs:\n"]
    asm = ["\t;;#ASMSTART\n", "\tv_mov_b32 v100, v3\n", "\t;;#ASMEND\n"]
    assert build.faults_in_assembly(head + asm + ["\tv_mov_b32_e32 v67, v3 ; v100\n"] + TAIL) == []
    for line in ("\tv_mov_b32_e32 v68, v3\n", "\tglobal_load_dwordx4 v[66:69], v3, s[0:1]\n"):
        assert len(build.faults_in_assembly(head + asm + [line] + TAIL)) == 1
    assert build.faults_in_assembly(HEAD + ["\tv_mov_b32_e32 v68, v3\n"] + TAIL) == []    # another kernel

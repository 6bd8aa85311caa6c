"""The build's check of the device assembly (CPU)."""
import glob
import os

import pytest

from paper_2105_10529_amd import check_asm

# a divergent branch with both sides: the lanes of one side jump to the join
# .LBB0_2, where the mask is flipped to the other side, and to .LBB0_4, where it
# is restored
BRANCH = """
kernel:
	s_and_saveexec_b64 s[8:9], vcc
	s_xor_b64 s[8:9], exec, s[8:9]
	s_cbranch_execz .LBB0_2
; %bb.1:
	v_mul_f64 v[0:1], v[2:3], v[2:3]
	v_accvgpr_write_b32 a5, v0
.LBB0_2:                                ;   in Loop: Header=BB0_9 Depth=1
{flip}	s_andn2_saveexec_b64 s[6:7], s[8:9]
	s_cbranch_execz .LBB0_4
; %bb.3:
	v_mov_b64_e32 v[0:1], v[4:5]
.LBB0_4:
{restore}	s_or_b64 exec, exec, s[6:7]
	v_accvgpr_write_b32 a0, v34
	s_endpgm
"""


@pytest.mark.parametrize("code", ["", "	s_mov_b32 s19, s80\n", "	v_readlane_b32 s4, v255, 12\n",
                                  "                                        ; implicit-def: $vgpr6\n"])
def test_joins_that_only_touch_the_mask_pass(code):
    assert check_asm.join_copies(BRANCH.format(flip=code, restore=code)) == []


@pytest.mark.parametrize("code", ["v_accvgpr_write_b32 a0, v34", "v_accvgpr_read_b32 v34, a0", "v_mov_b32_e32 v8, v3",
                                  "scratch_store_dword off, v34, off offset:16 ; 4-byte Folded Spill",
                                  "scratch_load_dword v34, off, off offset:16 ; 4-byte Folded Reload"])
def test_copies_ahead_of_the_masks_restore_are_found(code):
    at = "	s_mov_b32 s19, s80\n	" + code + "\n"
    found = check_asm.join_copies(BRANCH.format(flip=at, restore=""))
    assert [f[:2] for f in found] == [("kernel", ".LBB0_2")] and len(found[0][2]) == 1
    found = check_asm.join_copies(BRANCH.format(flip="", restore=at))
    assert [f[:2] for f in found] == [("kernel", ".LBB0_4")]
    assert len(check_asm.join_copies(BRANCH.format(flip=at, restore=at))) == 2


def test_other_blocks_are_left_alone():
    """The body of a side, and a label that is reached under the full mask."""
    text = """
kernel:
	s_cbranch_scc1 .LBB0_1
	s_andn2_saveexec_b64 s[4:5], s[4:5]
	s_cbranch_execnz .LBB0_2
.LBB0_1:
	v_accvgpr_read_b32 v23, a3
	s_and_saveexec_b64 s[4:5], vcc
	s_endpgm
.LBB0_2:
	v_mov_b64_e32 v[126:127], v[128:129]
	s_or_b64 exec, exec, s[4:5]
	s_endpgm
"""
    assert check_asm.join_copies(text) == []


def test_divergent_loops_are_counted():
    text = """
kernel:
.LBB0_1:
	s_andn2_b64 exec, exec, s[4:5]
	s_cbranch_execnz .LBB0_1
	s_endpgm
other:
	s_andn2_b64 s[0:1], exec, s[4:5]
	s_endpgm
"""
    assert check_asm.divergent_loops(text) == {"kernel": 1}


def test_the_integrand_kernels_have_no_divergent_loop():
    """Of the kernels that evaluate the amplitudes of listed points; they fill
    the register file, where divergent regions are where the compiler moves
    registers."""
    units = glob.glob(os.path.join(os.path.dirname(check_asm.__file__), "_build", "inst_*gfx950.s"))
    if not units:
        pytest.skip("the library was not built here")
    seen = 0
    for path in units:
        with open(path) as f:
            text = f.read()
        seen += text.count("11k_integrandILi") > 0
        assert [fn for fn in check_asm.divergent_loops(text) if "11k_integrandILi" in fn] == [], path
    assert seen >= 9

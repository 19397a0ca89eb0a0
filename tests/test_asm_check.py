"""The build's check of the generated assembly: per-lane instructions in front of
an exec restore are found where the lanes of a divergent region or loop meet again,
and the forms that are in order pass."""
import pytest

from paper_2102_02989_amd import asm_check, build

# a region skipped when no lane is active; the meeting block opens with {0}
REGION = """_Z6kernelPd:
; %bb.0:
\tv_cmp_gt_f64_e32 vcc, v[0:1], v[2:3]
\ts_and_saveexec_b64 s[18:19], vcc
\ts_cbranch_execz .LBB0_2
; %bb.1:
\tv_mul_f64 v[4:5], v[0:1], v[2:3]
.LBB0_2:                                ;   in Loop: Header=BB0_1 Depth=1
{0}\ts_or_b64 exec, exec, s[18:19]
\tv_add_f64 v[0:1], v[4:5], v[6:7]
\ts_endpgm
"""
LOOP = """_Z6kernelPd:
.LBB0_1:
\tv_add_f64 v[0:1], v[0:1], v[2:3]
\tv_cmp_gt_i32_e32 vcc, v8, v9
\ts_andn2_b64 exec, exec, vcc
\ts_cbranch_execnz .LBB0_1
; %bb.2:
{0}\ts_or_b64 exec, exec, s[18:19]
\ts_endpgm
"""
COPY = "\tv_accvgpr_write_b32 a6, v40\n\ts_mov_b32 s99, s37\n"


@pytest.mark.parametrize("text", [REGION, LOOP])
@pytest.mark.parametrize("before", [COPY, "\tscratch_store_dword off, v3, off offset:8 ; 4-byte Folded Spill\n",
                                    "\tscratch_load_dword v3, off, off offset:8 ; 4-byte Folded Reload\n",
                                    "\ts_mov_b32 s99, s37\n\tv_mov_b32_e32 v7, v8\n"])
def test_found(text, before):
    n, found = asm_check.check(text.format(before))
    assert n == 1 and len(found) == 1
    assert found[0][0] == "_Z6kernelPd" and found[0][2].split()[0] in before


@pytest.mark.parametrize("text", [REGION, LOOP])
@pytest.mark.parametrize("before", ["", "\ts_mov_b32 s99, s37\n", "\tv_writelane_b32 v250, s12, 7\n",
                                    "\tv_readlane_b32 s12, v250, 7\n"])
def test_passes(text, before):
    assert asm_check.check(text.format(before)) == (1, [])


def test_region_out_of_line_passes():
    """A region entered by a branch ends with the restore: its work is its own."""
    text = """_Z6kernelPd:
\ts_and_saveexec_b64 s[0:1], vcc
\ts_cbranch_execnz .LBB0_9
.LBB0_8:
\ts_endpgm
.LBB0_9:
\tv_mov_b32_e32 v1, v2
\tglobal_store_dword v0, v1, s[2:3]
\ts_or_b64 exec, exec, s[0:1]
\ts_branch .LBB0_8
"""
    assert asm_check.check(text) == (0, [])


def test_build_refuses(tmp_path):
    f = tmp_path / "k.s"
    f.write_text(REGION.format(COPY))
    with pytest.raises(RuntimeError, match="v_accvgpr_write_b32 a6, v40"):
        build.check_assembly(str(f))
    f.write_text(REGION.format(""))
    assert build.check_assembly(str(f)) == 1
    f.write_text("nothing that the check reads\n")
    with pytest.raises(RuntimeError, match="no exec restore"):
        build.check_assembly(str(f))

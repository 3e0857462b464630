"""The build refuses a code of the planes-in-registers kernels in which the compiler touches the registers that their asm blocks number."""
import pytest

from paper_1908_05460_amd import build

ASM = """_ZN5wgrad18approx_gather_regsENS_9RegsMultiE: ; @approx_gather_regs, v99 in a comment
\tv_add_u32_e32 v3, s12, v{high}
\tds_read_b128 v[{low}:{high}], v2
\t;;#ASMSTART
\tv_fmac_f32 v[19+9*7+3], s3, v[55]
\t;;#ASMEND
{extra}
\t.amdhsa_kernel _ZN5wgrad18approx_gather_regsENS_9RegsMultiE
\t.end_amdhsa_kernel
"""


def asm(high, extra=""):
    return ASM.format(high=high, low=high - 3, extra=extra)


def test_layouts_name_their_first_register():
    assert build.numbered_registers() == {"approx_gather_regs": 19, "approx_gather_regs8": 61}


def test_code_within_its_registers_passes():
    build.check_numbered_registers(asm(18), {"approx_gather_regs": 19})


@pytest.mark.parametrize("text", [asm(19), asm(126), asm(18, "\tv_accvgpr_write_b32 a0, v3"), asm(18, "\tscratch_store_dword off, v3, s32"), "nothing"])
def test_code_beyond_them_is_refused(text):
    with pytest.raises(RuntimeError):
        build.check_numbered_registers(text, {"approx_gather_regs": 19})

"""The checks of test_isa_checks.py on the kernels of short calls, which have a source of their own."""
import re

import pytest

from tests import test_isa_checks as T

pytestmark = T.pytestmark


@pytest.fixture(scope="module")
def source(tmp_path_factory):
    # lists of 4 and 12 with and without a bias, 20 without; d whole stages or not
    return T.assembly("ll_project_short", tmp_path_factory.mktemp("isa")), "ll_lens_gemm_short_kernel", 10


def test_short_kernels(source):
    T.test_m0_is_only_written_by_the_lds_base_setter(source)
    T.test_projection_kernels_fit_one_wave_per_simd_without_scratch(source)
    T.test_no_valu_reads_an_sgpr_a_valu_wrote_within_two_instructions(source)
    T.test_list_insertions_are_eight_byte_instructions_on_their_boundaries(source)


def test_the_epilogues_are_placed(source):
    """Their code, of a whole tile and of half a tile, starts 4 bytes past a multiple of 32, whatever stands before it."""
    asm, kernel, count = source
    found = [len(re.findall(r"\.p2align\s+5\s+s_nop 0\s+;;#ASMEND", m.group(1)))
             for m in re.finditer(r"^_Z\w*" + kernel + r"\w*:[^\n]*\n(.*?)\n\s*s_endpgm", asm, re.S | re.M)]
    assert found == [2] * count

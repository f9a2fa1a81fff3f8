"""The checks of test_isa_checks.py on the kernels of short calls, which have a source of their own."""
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

"""The checks of test_isa_checks.py on the sweeps that form u themselves, which have a source of their own."""
import pytest

from tests import test_isa_checks as T

pytestmark = T.pytestmark


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    parts = T.assembly("ll_project_sweep", tmp_path_factory.mktemp("isa")).split(".Lfunc_end")
    return "\n\ts_endpgm\n.Lfunc_end".join(x.replace("s_endpgm", "s_nop 0") for x in parts)   # (a body's first end is the way out of the form not taken)


# the arg max of whole K stages; of ragged ones, lists, and the two general forms
@pytest.mark.parametrize("kernel,count,factored", [("ll_lens_gemm_dma_kernel", 1, 1), ("ll_lens_gemm_dma_tail_kernel", 4, 2)])
def test_whole_sweeps(asm, kernel, count, factored):
    T.test_m0_is_only_written_by_the_lds_base_setter((asm, kernel, count))
    T.test_projection_kernels_fit_one_wave_per_simd_without_scratch((asm, kernel, count))
    products = broadcasts = 0
    for name, ins in T.kernel_bodies(asm, kernel).items():
        ins = [l for l in (l.split(";")[0].strip() for l in ins) if l]
        assert not any(l.startswith("flat_") for l in ins), name      # the tables are read as LDS
        for i, l in enumerate(ins):
            product = l.startswith("v_mfma_f32_16x16x4_f32")
            if not product and not l.startswith("v_subrev_f32_dpp"):
                continue
            operands = l.split(None, 1)[1].split(",")
            reads = set().union(*(T.registers(o) for o in operands[1:])) if product else T.registers(operands[1])
            states, j = 0, i - 1
            while j >= 0 and states < 2:
                assert ins[j].startswith("v_mfma") or not T.written(ins[j]) & reads, (name, ins[j], l)
                states += T.wait_states(ins[j])
                j -= 1
            broadcasts += not product
            products += product
            states, j = 0, i + 1
            while product and j < len(ins) and states < 18:
                if ins[j].startswith(("v_", "global_", "ds_")) and not ins[j].startswith("v_mfma") and " " in ins[j]:
                    touched = set().union(*(T.registers(o) for o in ins[j].split(None, 1)[1].split(",")))
                    assert not touched & T.registers(operands[0]), (name, l, ins[j])
                states += T.wait_states(ins[j])
                j += 1
    assert products == 32 * factored and broadcasts == 10 * factored   # (no second table: no product of its own)

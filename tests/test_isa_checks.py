"""Checks on the compiled device code of the projection kernels (no GPU needed: hipcc cross-compiles).

The direct-to-LDS kernel sets M0 (the LDS base of its load-to-LDS instructions) once per operand
tile and relies on it staying put until the tile's last load; it also sizes its register use to
exactly one wavefront per SIMD with no scratch.  Both are properties of the generated code, not
of the source, so they are checked on the assembly.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_06483_amd", "csrc")
# source, its direct-to-LDS kernels, and how many there are
SOURCES = {
    "ll_project": ("ll_lens_gemm_dma_kernel", 10),             # four top-k list lengths, each with and without a bias, and the two steering sweeps
    "ll_project_tail": ("ll_lens_gemm_dma_tail_kernel", 11),   # ragged hidden sizes: the same but the longest list with a bias; the two general sweeps
}

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")


def assembly(name, directory):
    out = directory / (name + ".s")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-S", "--cuda-device-only",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, name + ".hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return out.read_text()


@pytest.fixture(scope="module", params=sorted(SOURCES))
def source(request, tmp_path_factory):
    """(assembly, name of the direct-to-LDS kernels in it, their number)"""
    return (assembly(request.param, tmp_path_factory.mktemp("isa")), *SOURCES[request.param])


def kernel_bodies(asm_text, needle):
    """{symbol: [instruction lines]} for every kernel whose mangled name contains `needle`."""
    bodies = {}
    for m in re.finditer(r"^(_Z\w*" + needle + r"\w*):[^\n]*\n(.*?)\n\s*s_endpgm", asm_text, re.S | re.M):
        lines = [l.strip() for l in m.group(2).splitlines()]
        bodies[m.group(1)] = [l for l in lines if l and not l.startswith((";", ".", "//")) and not l.endswith(":")]
    return bodies


def test_m0_is_only_written_by_the_lds_base_setter(source):
    asm, kernel, count = source
    bodies = kernel_bodies(asm, kernel)
    assert len(bodies) == count, sorted(bodies)
    for name, ins in bodies.items():
        loads = [i for i, l in enumerate(ins) if l.startswith("global_load_lds_dwordx4")]
        assert len(loads) >= 16 + 36, (name, len(loads))          # main loop + prologue
        for i, l in enumerate(ins):
            if "m0" not in l.split(";")[0]:
                continue
            # the only mention of M0: "s_mov_b32 m0, sN" and the wait state that follows it
            assert re.fullmatch(r"s_mov_b32 m0, s\d+", l.split(";")[0].strip()), (name, l)
            assert ins[i + 1].startswith("s_nop"), (name, ins[i + 1])
        # nothing that implicitly uses M0 (indexed register moves, messages, GWS)
        for l in ins:
            op = l.split()[0]
            assert not op.startswith(("v_movrel", "s_movrel", "s_sendmsg", "ds_gws", "s_set_gpr_idx")), (name, l)


def test_projection_kernels_fit_one_wave_per_simd_without_scratch(source):
    asm, kernel, count = source
    meta = {}
    for m in re.finditer(r"\.name:\s+(\S+)\n(.*?)\.wavefront_size", asm, re.S):
        block = m.group(2)
        get = lambda key: int(re.search(r"\." + key + r":\s+(\d+)", block).group(1))
        meta[m.group(1)] = dict(vgpr=get("vgpr_count"), scratch=get("private_segment_fixed_size"),
                                vspill=get("vgpr_spill_count"))
    dma = {k: v for k, v in meta.items() if kernel in k}
    assert len(dma) == count
    for name, v in dma.items():
        assert v["vgpr"] <= 512 and v["scratch"] == 0 and v["vspill"] == 0, (name, v)


def test_no_valu_reads_an_sgpr_a_valu_wrote_within_two_instructions(source):
    """gfx950 needs two wait states between a VALU instruction that writes an SGPR (a comparison,
    a carry-out) and a VALU instruction that reads it.  The compiler keeps that distance for its
    own instructions but does not look inside inline asm: check the hand-written selects and
    add-with-carry of the top-k epilogue."""
    asm, kernel, _ = source
    bodies = {**kernel_bodies(asm, kernel), **kernel_bodies(asm, "ll_lens_gemm_kernel")}
    assert bodies
    checked = 0
    for name, ins in bodies.items():
        ins = [l.split(";")[0].strip() for l in ins]
        ins = [l for l in ins if l]
        for i, l in enumerate(ins):
            m = re.fullmatch(r"v_cndmask_b32 v\d+, v\d+, v\d+, (s\[\d+:\d+\])", l) or \
                re.fullmatch(r"v_addc_co_u32_e64 v\d+, s\[\d+:\d+\], v\d+, v\d+, (s\[\d+:\d+\])", l)
            if not m:
                continue
            checked += 1
            sreg = m.group(1)
            for prev in ins[max(0, i - 2):i]:
                ops = prev.split(None, 1)
                if len(ops) == 2 and ops[0].startswith("v_"):
                    dests = ops[1].split(",")[:2]            # destination, and carry-out where there is one
                    assert all(sreg != dd.strip() for dd in dests), (name, prev, l)
    assert checked > 1000


def test_list_insertions_are_eight_byte_instructions_on_their_boundaries(source):
    """Four slots of a list are sixteen instructions of eight bytes, which take 3 to 4 % longer (whole calls of lists of 24) from four
    bytes off: each such block starts at an alignment directive, and none holds another instruction."""
    asm, kernel, _ = source
    blocks = 0
    for m in re.finditer(r"^(_Z\w*(?:" + kernel + r"|ll_lens_gemm_kernel)\w*TopKEpilogueILi\d+E\w*):[^\n]*\n(.*?)\n\s*s_endpgm", asm, re.S | re.M):
        lines = [l.split(";")[0].strip() for l in m.group(2).splitlines()]
        lines = [l for l in lines if l]
        starts = [i for i, l in enumerate(lines) if l.split() == [".p2align", "3"]]
        assert sum(l.startswith("v_med3_f32") for l in lines) == 4 * len(starts), m.group(1)
        for i in starts:
            body = lines[i + 1:i + 17]
            assert all(re.match(r"v_(cmp_gt_f32_e64|med3_f32|cndmask_b32_e64) ", l) for l in body), (m.group(1), body)
        blocks += len(starts)
    assert blocks > 0


LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-mc")), reason="no assembler")
def test_the_k_loop_of_projections_without_a_bias_starts_at_byte_44_of_a_line(tmp_path):
    text = assembly("ll_project", tmp_path)
    obj = tmp_path / "ll_project.o"
    subprocess.run([os.path.join(LLVM, "llvm-mc"), "-triple=amdgcn-amd-amdhsa", "-mcpu=gfx950", "-filetype=obj", "-o", str(obj)],
                   input=text, text=True, check=True)
    found = {}
    listing = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--mcpu=gfx950", str(obj)], capture_output=True, text=True, check=True).stdout
    for m in re.finditer(r"^[0-9a-f]+ <(_Z\w*ll_lens_gemm_dma_kernel\w*TopKEpilogueILi(\d+)ELb0E\w*)>:\n(.*?)(?=\n\n)", listing + "\n\n", re.S | re.M):
        at = [int(x, 16) for x in re.findall(r"v_mfma_f32_16x16x32_bf16[^\n]*//\s*([0-9A-F]+):", m.group(3))]
        assert len(at) == 256                             # a tile's first stage and the loop's
        found[int(m.group(2))] = at[128] % 64
    assert found == {4: 44, 12: 44, 20: 44, 32: 44}


def test_the_general_sweeps_groups_are_placed(source):
    """Their code starts 20 bytes past a multiple of 32, whatever stands before it."""
    asm, kernel, _ = source
    for m in re.finditer(r"^(_Z\w*" + kernel + r"\w*SweepEpilogueILi\dELb1E\w*):[^\n]*\n(.*?)\n\s*s_endpgm", asm, re.S | re.M):
        assert len(re.findall(r"\.p2align\s+5\s+(?:s_nop 0\s+){5};;#ASMEND", m.group(2))) == 1, m.group(1)


def registers(operand):
    """The vector registers that an operand names."""
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand.strip())
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def written(instruction):
    return registers(instruction.split(None, 1)[1].split(",")[0]) if instruction.startswith("v_") and " " in instruction else set()


def wait_states(instruction):
    nop = re.fullmatch(r"s_nop (\d+)", instruction)
    if instruction.startswith("v_mfma_f32_16x16x4"):
        return 8                                          # passes of four cycles
    return 1 + int(nop.group(1)) if nop else 1


def test_the_sweeps_products_and_broadcasts_keep_their_distances(source):
    """The steering sweep writes its fp32 matrix products and its DPP broadcasts as instructions, whose hazards the compiler does not
    see: two wait states between a vector instruction that writes an operand and the product or the DPP instruction that reads it,
    and 18 between a product and a vector or memory instruction that touches its result."""
    asm, kernel, _ = source
    products = broadcasts = 0
    for name, ins in kernel_bodies(asm, kernel + r"\w*SweepEpilogue").items():
        ins = [l.split(";")[0].strip() for l in ins]
        ins = [l for l in ins if l]
        for i, l in enumerate(ins):
            product = l.startswith("v_mfma_f32_16x16x4_f32")
            if not product and not l.startswith("v_subrev_f32_dpp"):
                continue
            operands = l.split(None, 1)[1].split(",")
            reads = set().union(*(registers(o) for o in operands[1:])) if product else registers(operands[1])
            states, j = 0, i - 1
            while j >= 0 and states < 2:
                assert ins[j].startswith("v_mfma") or not written(ins[j]) & reads, (name, ins[j], l)
                states += wait_states(ins[j])
                j -= 1
            if not product:
                broadcasts += 1
                continue
            products += 1
            result = registers(operands[0])
            states, j = 0, i + 1
            while j < len(ins) and states < 18:
                if ins[j].startswith(("v_", "global_", "ds_")) and not ins[j].startswith("v_mfma") and " " in ins[j]:
                    touched = set().union(*(registers(o) for o in ins[j].split(None, 1)[1].split(",")))
                    assert not touched & result, (name, l, ins[j])
                states += wait_states(ins[j])
                j += 1
    assert products == 96 and broadcasts == 20            # two kernels of 48 products; nine limits and a spread, in each

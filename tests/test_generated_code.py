"""What assembly blocks ask of the code around them, which the compiler does not look into, in the code of every kernel (CPU)."""
import re

import pytest

import _asm


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    from paper_2311_02382_amd import build
    return _asm.assembly(tmp_path_factory.mktemp("asm"), build.SOURCES)


def test_loads_from_a_scalar_base_wait_for_the_vector_instruction_that_wrote_it(code):
    # A vector-memory instruction may read a scalar register that a vector instruction (v_readfirstlane, a comparison, a carry) wrote
    # five wait states later at the earliest
    seen = 0
    for source, text in code.items():
        for name, lines in _asm.kernels(text).items():
            flow = _asm.Flow(lines)
            for i, line in enumerate(flow.code):
                if not line.startswith(("global_", "buffer_", "flat_", "scratch_")):
                    continue
                base = {r for r in set().union(*_asm.operands(line)) if r[0] in ("s", "vcc")}
                seen += line.startswith("global_load_lds")
                for before, waited in flow.within(i, 5) if base else ():
                    assert not (before.startswith("v_") and _asm.written(before) & base), (source, name, before, waited, line)
    assert seen > 1000


def test_feed_forward_epilogues_have_two_wavefronts_per_simd(code):
    # GeLU is vector work behind the contraction: a wavefront alone on its SIMD, as in the wide tiles, issues it at half the rate
    names = [name for name in _asm.kernels(code["lss_proj.hip"]) if "proj_" in name and not name.endswith("ELi0EEEvNS0_8ProjArgsE")]
    assert len(names) == 14 and not [name for name in names if "GemmWide" in name]


def test_wide_tiles_accumulators_belong_to_matrix_instructions(code):
    # They are cleared, summed up and read, never copied (a lone wavefront takes 0.8 us to go over them); and since their matrix instructions are assembly, along every
    # path: no vector instruction writes an operand within two wait states ahead, no other kind of matrix instruction an accumulator and nothing else
    # touches one within twenty behind it (the longest that any matrix instruction of the architecture asks for).
    wide = 0
    for name, lines in _asm.kernels(code["lss_proj.hip"]).items():
        if "GemmWide" not in name:
            continue
        wide += 1
        flow = _asm.Flow(lines)
        products = [i for i, line in enumerate(flow.code) if line.startswith("v_mfma")]
        assert not [x for x in flow.code[products[0]:products[-1]] if x.startswith(("v_accvgpr_write", "v_accvgpr_mov"))], name
        for i, line in enumerate(flow.code):
            op, used = line.split()[0], set().union(*_asm.operands(line))
            if op.startswith("v_mfma"):
                for before, waited in flow.within(i, 2):
                    assert not (before.startswith("v_") and not before.startswith("v_mfma") and _asm.written(before) & used), (name, before, waited, line)
            acc = {r for r in used if r[0] == "a"}
            for before, waited in flow.within(i, 20) if acc else ():
                if before.startswith("v_mfma") and before.split()[0] != op:
                    assert not _asm.written(before) & acc, (name, before, waited, line)
    assert wide == 5


def test_products_keep_their_registers(code):
    # (the float weight gradient in wide tiles had one in scratch memory: 512 registers are all there are)
    sizes = re.findall(r"\.amdhsa_kernel (\S+).*?\.amdhsa_private_segment_fixed_size (\d+)", code["lss_proj.hip"], re.S)
    assert len(sizes) == len(_asm.kernels(code["lss_proj.hip"])) and not [name for name, size in sizes if size != "0"]


def test_scalar_register_m0_belongs_to_assembly_blocks(code):
    # The direct loads set it and do not restore it
    seen = 0
    for source, text in code.items():
        inside = False
        for line in text.splitlines():
            inside = "#ASMSTART" in line or inside and "#ASMEND" not in line
            if re.match(r"\t[a-z]", line) and re.search(r"\bm0\b", line):
                seen += 1
                assert inside, (source, line)
    assert seen > 1000

"""What assembly blocks ask of the code around them, which the compiler does not look into, in the code of every kernel (CPU)."""
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

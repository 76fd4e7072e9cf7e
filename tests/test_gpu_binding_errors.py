"""What the binding says when tensors do not fit or do not exist."""
import pytest
import torch

from paper_2311_02382_amd import lss

pytestmark = pytest.mark.gpu


def _t(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype, device="cuda")


@pytest.mark.parametrize("given,message", [((2, 9, 64), r"output has shape \(2, 9, 64\), expected \(2, 8, 64\)"),
                                           ((1024,), r"output has shape \(1024,\), expected \(2, 8, 64\)")])
def test_a_wrong_output_names_both_shapes(given, message):
    with pytest.raises(ValueError, match=message):
        lss.lss_gelu_fwd(_t(2, 8, 64), g=_t(*given))


def test_out_of_memory_keeps_its_type():
    # the outputs of 10^11 rows (25 TB) are asked for before the library sees the call
    with pytest.raises(torch.OutOfMemoryError):
        lss.lss_project_qkv(_t(1, 8, 128), _t(128, 128), _t(128, 256), 0, 10 ** 11, 2)
    torch.cuda.synchronize()


def test_other_errors():
    with pytest.raises(ValueError, match="u must be a contiguous torch.bfloat16 device tensor"):
        lss.lss_gelu_fwd(_t(2, 64, dtype=torch.float32))
    with pytest.raises(TypeError, match="expected a torch tensor, got list"):
        lss.lss_gelu_fwd([1.0])
    with pytest.raises(lss.LssError, match="LSS_ERR_SHAPE") as e:
        lss.lss_gelu_fwd(_t(12))
    assert e.value.code == -2
    with pytest.raises(ValueError, match="workspace of 16 bytes, need"):
        lss.lss_segment_attn_fwd(_t(1, 8, 1, 64), _t(1, 8, 1, 64), _t(1, 8, 1, 64), 0, workspace=_t(16, dtype=torch.uint8))

"""The plain C entry points on the GPU, called without the binding's native half: registered workspace, raw pointers."""
import pytest
import torch

from paper_2311_02382_amd import lss
from _util import stage_all

pytestmark = pytest.mark.gpu

B, L_X, H, S0, L_S = 1, 900, 3, 400, 200


def _p(t):
    return t.data_ptr()


def _problem(kind, d=64):
    Q, K, V, DO = stage_all(B, L_X, H, d, 9300 + d, kind)
    sl = slice(S0, S0 + L_S)
    return Q.dev[:, sl].contiguous(), K.dev, V.dev, DO.dev[:, sl].contiguous()


def _fresh(q, k):
    return (torch.full_like(q, 3.0), torch.full((B, H, L_S), 3.0, device="cuda"), torch.full_like(q, 3.0),
            torch.full(k.shape, 3.0, device="cuda"), torch.full(k.shape, 3.0, device="cuda"))


def _same(got, want):
    for name, a, b in zip(("out", "lse", "dq", "dk_partial", "dv_partial"), got, want):
        assert torch.equal(a, b), name


def _want(q, k, v, do, **drop):
    out, lse = lss.lss_segment_attn_fwd(q, k, v, S0, True, **drop)
    return (out, lse, *lss.lss_segment_attn_bwd(q, k, v, S0, out, lse, do, True, **drop))


def test_a_call_of_the_binding_registers_its_workspace_again():
    q, k, v, do = _problem("bf16")
    want = _want(q, k, v, do)
    lib = lss.load()
    out, lse, *_ = _fresh(q, k)
    args = (_p(q), _p(k), _p(v), S0, L_S, L_X, B, H, 64, 1, _p(out), _p(lse), torch.cuda.current_stream().cuda_stream)
    lss.lss_set_workspace(None)
    assert lib.lss_segment_attn_fwd(*args) == -6
    lss.lss_segment_attn_fwd(q, k, v, S0, True)         # (no new buffer: an earlier call's is large enough)
    assert lib.lss_segment_attn_fwd(*args) == 0
    assert torch.equal(out, want[0]) and torch.equal(lse, want[1])

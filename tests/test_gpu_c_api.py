"""The plain C entry points on the GPU, called without the binding's native half: registered workspace, raw pointers."""
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, rel_err, stage_all, to_np

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


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["bf16", "f32"])
def test_plain_and_dropout_calls_equal_the_bindings(kind, d):
    # lss_segment_attn_fwd / _bwd, their _f32 twins and the _dropout pair: the buffer registered for the GPU, results bit for
    # bit those of the general forms that the binding calls
    q, k, v, do = _problem(kind, d)
    lib = lss.load()
    st = torch.cuda.current_stream().cuda_stream
    shape = (S0, L_S, L_X, B, H, d, 1)
    eb = 4 if kind == "f32" else 2
    need = lib.lss_workspace_bytes(L_S, L_X, B, H, d, eb)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    suffix = "_f32" if kind == "f32" else ""
    try:
        for drop in ({}, dict(p_drop=0.0, seed=3), dict(p_drop=0.15, seed=12345678901)):
            want = _want(q, k, v, do, **drop)
            out, lse, dq, dk, dv = got = _fresh(q, k)
            lss.lss_set_workspace(ws)
            head, tail = (_p(q), _p(k), _p(v), *shape), (_p(out), _p(lse), _p(do), _p(dq), _p(dk), _p(dv), st)
            if drop:
                more = (drop["p_drop"], drop["seed"], eb)
                assert lib.lss_segment_attn_fwd_dropout(*head, *more, _p(out), _p(lse), st) == 0
                assert lib.lss_segment_attn_bwd_dropout(*head, *more, *tail) == 0
            else:
                assert getattr(lib, "lss_segment_attn_fwd" + suffix)(*head, _p(out), _p(lse), st) == 0
                assert getattr(lib, "lss_segment_attn_bwd" + suffix)(*head, *tail) == 0
            torch.cuda.synchronize()
            _same(got, want)
    finally:
        torch.cuda.synchronize()
        lss.lss_set_workspace(None)


def test_an_empty_segment_writes_zero_partials_through_the_plain_calls():
    _, k, v, _ = _problem("bf16")
    lib = lss.load()
    st = torch.cuda.current_stream().cuda_stream
    for name in ("lss_segment_attn_bwd", "lss_segment_attn_bwd_f32", "lss_segment_attn_bwd_noalloc"):
        dk, dv = (torch.full(k.shape, 3.0, device="cuda") for _ in range(2))
        assert getattr(lib, name)(None, _p(k), _p(v), S0, 0, L_X, B, H, 64, 1, None, None, None, None, _p(dk), _p(dv), st) == 0
        assert torch.count_nonzero(dk) == 0 and torch.count_nonzero(dv) == 0


def test_plain_projection_backward_equals_the_bindings():
    torch.manual_seed(5)
    h, d = 2, 64
    e = h * d
    dq = torch.randn(B, L_S, h, d, device="cuda").bfloat16()
    dk, dv = (torch.randn(B, L_X, h, d, device="cuda") for _ in range(2))
    wq, wkv = torch.randn(e, e, device="cuda").bfloat16(), torch.randn(e, 2 * e, device="cuda").bfloat16()
    rows = S0 + L_S
    want = lss.lss_project_bwd(dq, dk, dv, wq, wkv, rows)
    dx_q, dx_p = torch.full((B, L_S, e), 3.0, device="cuda"), torch.full((B, L_X, e), 3.0, device="cuda")
    assert lss.load().lss_project_bwd(_p(dq), _p(dk), _p(dv), _p(wq), _p(wkv), L_S, L_X, rows, B, h, d, _p(dx_q), _p(dx_p),
                                      torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(dx_q, want[0]) and torch.equal(dx_p, want[1])


@pytest.mark.parametrize("l_s", [58, 128])
def test_a_workspace_sized_for_bf16_partial_results_still_serves(l_s):
    # one head, up to 16 key splits: their partial outputs took two bytes per element, and callers have buffers of that size
    l_x, d, s0, splits = 8192, 64, 8000, 16
    Q, K, V, DO = stage_all(1, l_x, 1, d, 9400 + l_s, "bf16")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    former = lss.lss_workspace_bytes(l_s, l_x, 1, 1, d) - splits * l_s * d * 2      # (a multiple of 256: no rounding between the regions)
    ro, rl = oracle.segment_fwd(Q.f64[:, sl], K.f64, V.f64, s0, True)
    ref = oracle.segment_bwd(Q.f64[:, sl], K.f64, V.f64, DO.f64[:, sl], s0, True)
    ws = torch.full((former + 256,), 7, dtype=torch.uint8, device="cuda")
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, workspace=ws[:former])
    grads = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, workspace=ws[:former])
    for a, b in zip((out, *grads), (ro, *ref)):
        assert rel_err(to_np(a), b) <= TOL["bf16"]["t"]
    assert torch.all(ws[former:] == 7)
    with pytest.raises(ValueError, match="need"):
        lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, workspace=ws[:former - 1])

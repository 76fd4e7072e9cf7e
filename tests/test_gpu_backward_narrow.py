"""The d = 128 backward on both sides of the rule for wavefronts of 16 rows: sizes at which a wavefront has no row or key, one,
or all of them, keys split or not, start values computed in the workgroup or before."""
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, bwd_plan, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, s0, l_s, causal
    (1, 129, 1, 0, 129, True), (1, 200, 2, 7, 81, True), (1, 320, 2, 0, 97, False), (2, 500, 1, 100, 257, True),
    (1, 1100, 2, 500, 600, True), (1, 900, 1, 0, 900, False), (1, 2000, 2, 1500, 113, True),
    (1, 1024, 64, 0, 1024, True), (1, 1025, 64, 0, 1025, True),     # 32 walks per compute unit, and more
]


@pytest.mark.parametrize("p_drop", [0.0, 0.25])
@pytest.mark.parametrize("B,l_x,H,s0,l_s,causal", SHAPES)
def test_backward_against_the_oracle(B, l_x, H, s0, l_s, causal, p_drop):
    plan = bwd_plan(B, l_x, H, 128, s0, l_s, causal, p_drop > 0)
    assert plan.narrow == (l_x != 1025) and plan.own == (l_x == 320)
    Q, K, V, DO = stage_all(B, l_x, H, 128, 7700 + l_x + l_s, "bf16")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    drop = {"p_drop": p_drop, "seed": 78} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, causal, **drop)
    grads = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    heads = slice(0, 2 if B == 1 else H)                # (one batch's heads do not depend on each other: two are enough to compare)
    args = (Q.f64[:, sl, heads], K.f64[:, :, heads], V.f64[:, :, heads], DO.f64[:, sl, heads], s0, causal)
    ref = oracle.segment_bwd_dropout(*args, p_drop, 78) if p_drop else oracle.segment_bwd(*args)
    for name, got, want in zip(("dq", "dk", "dv"), grads, ref):
        assert rel_err(to_np(got)[:, :, heads], want) <= TOL["bf16"]["t"], name
    again = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))

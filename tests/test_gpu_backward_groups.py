"""Backward workgroups of one and of two groups of wavefronts, the latter with half the key or query tiles each: sizes at which the
second group has no tile, one, a partial one or one less than the first, start values computed in the workgroup or before, keys
split or not."""
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, bwd_plan, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, s0, l_s, causal
    (1, 129, 1, 0, 129, True), (1, 200, 2, 7, 193, True), (1, 320, 2, 0, 320, False), (2, 500, 1, 100, 257, True),
    (1, 700, 2, 0, 577, True), (1, 1100, 2, 500, 600, True), (1, 64, 1, 0, 64, True), (1, 900, 2, 0, 900, False),
    (1, 2000, 2, 1500, 300, True),                                                      # keys split besides
]


# Two groups: start values in the workgroup or before, keys split or not
TWO_GROUPS = [  # B, l_x, H, s0, l_s, causal, p_drop, (own, split)
    (1, 892, 1, 609, 283, True, 0.0, (1, False)), (3, 2569, 4, 609, 390, True, 0.0, (1, False)),
    (1, 897, 2, 640, 257, True, 0.0, (1, False)), (1, 1025, 1, 576, 449, True, 0.0, (1, False)),     # last key tile: one query tile, of the first group
    (1, 276, 6, 64, 171, True, 0.25, (1, False)), (1, 257, 2, 64, 193, True, 0.25, (1, False)),      # (the second here too)
    (1, 1961, 1, 1536, 389, True, 0.0, (1, True)), (1, 14265, 8, 2176, 346, True, 0.0, (1, True)),
    (1, 1677, 3, 1449, 162, True, 0.25, (1, True)), (1, 1587, 4, 1381, 206, False, 0.25, (1, True)),
    (1, 17417, 1, 7155, 241, False, 0.0, (1, True)), (1, 17417, 1, 7155, 241, False, 0.25, (1, True)),       # 16 ranges
    (1, 325, 1, 0, 325, True, 0.0, (0, False)), (1, 513, 2, 0, 513, True, 0.0, (0, False)),         # first query tile: two key tiles
    (1, 325, 1, 0, 325, True, 0.25, (0, False)), (1, 513, 2, 0, 513, True, 0.25, (0, False)),
    (1, 1232, 1, 894, 338, True, 0.0, (0, True)), (1, 1153, 2, 832, 321, True, 0.0, (0, True)),
    (1, 1232, 1, 894, 338, True, 0.25, (0, True)), (1, 1153, 2, 832, 321, True, 0.25, (0, True)),
]


def check(B, l_x, H, s0, l_s, causal, p_drop):
    Q, K, V, DO = stage_all(B, l_x, H, 64, 9400 + l_x + l_s, "bf16")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    drop = {"p_drop": p_drop, "seed": 78} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, causal, **drop)
    grads = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    args = (Q.f64[:, sl], K.f64, V.f64, DO.f64[:, sl], s0, causal)
    ref = oracle.segment_bwd_dropout(*args, p_drop, 78) if p_drop else oracle.segment_bwd(*args)
    for name, got, want in zip(("dq", "dk", "dv"), grads, ref):
        assert rel_err(to_np(got), want) <= TOL["bf16"]["t"], name
    again = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))
    # a gradient written over the forward's output: D from a launch of its own
    over = out.clone()
    dq, dk, dv = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, over, lse, do, causal, dq=over, **drop)
    for name, got, want in zip(("dq", "dk", "dv"), (dq, dk, dv), ref):
        assert rel_err(to_np(got), want) <= TOL["bf16"]["t"], name


@pytest.mark.parametrize("p_drop", [0.0, 0.25])
@pytest.mark.parametrize("B,l_x,H,s0,l_s,causal", SHAPES)
def test_backward_against_the_oracle(B, l_x, H, s0, l_s, causal, p_drop):
    check(B, l_x, H, s0, l_s, causal, p_drop)


@pytest.mark.parametrize("B,l_x,H,s0,l_s,causal,p_drop,form", TWO_GROUPS)
def test_two_groups_against_the_oracle(B, l_x, H, s0, l_s, causal, p_drop, form):
    plan = bwd_plan(B, l_x, H, 64, s0, l_s, causal, p_drop > 0)
    assert plan.groups == 2 and not plan.one_pass and (plan.own, plan.splits > 1) == form
    check(B, l_x, H, s0, l_s, causal, p_drop)

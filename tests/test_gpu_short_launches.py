"""Forms that short launches at d = 64 take: forward workgroups of four groups of wavefronts (32 or 64 query rows), backward ones of eight
wavefronts of 16 rows.  Sizes at which groups have no key tile, one or a partial one, rows and keys of the last wavefronts do not exist, and
the launch just fits the chip."""
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, bwd_plan, fwd_plan, lse_err, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

FORWARD = [  # B, l_x, H, s0, l_s, causal, p_drop, (row blocks, groups, split)
    (1, 75, 9, 0, 75, True, 0.0, (1, 4, False)), (1, 33, 17, 0, 33, False, 0.0, (1, 4, False)), (1, 193, 5, 60, 129, True, 0.0, (1, 4, False)),
    (1, 700, 5, 256, 256, True, 0.0, (1, 4, False)), (1, 700, 16, 0, 497, True, 0.0, (1, 4, False)), (2, 1377, 4, 705, 301, True, 0.0, (1, 4, False)),
    (2, 1500, 8, 923, 577, True, 0.0, (2, 4, False)),
    (2, 2113, 8, 1024, 1000, True, 0.0, (2, 4, False)), (1, 4100, 16, 3070, 1024, True, 0.0, (2, 4, False)),
    (1, 190, 9, 90, 100, True, 0.25, (1, 4, False)), (1, 193, 5, 60, 129, False, 0.25, (1, 4, False)), (1, 700, 12, 100, 420, True, 0.25, (1, 4, False)),
    (2, 2113, 8, 1024, 1000, True, 0.25, (2, 4, False)), (1, 4100, 16, 3070, 1024, True, 0.25, (2, 4, False)),
]
BACKWARD = [  # B, l_x, H, s0, l_s, causal, p_drop, (own, split)
    (1, 75, 3, 0, 75, True, 0.0, (1, False)), (1, 193, 5, 60, 129, True, 0.0, (1, False)), (1, 129, 2, 0, 128, False, 0.0, (1, False)),
    (1, 1024, 4, 768, 256, True, 0.0, (1, True)), (1, 3000, 2, 2500, 81, True, 0.0, (1, True)),
    (1, 454, 2, 130, 289, True, 0.0, (0, False)), (1, 475, 1, 29, 276, True, 0.0, (0, False)), (1, 500, 4, 7, 65, False, 0.25, (1, True)),
    (1, 193, 5, 60, 128, True, 0.25, (1, False)), (1, 1500, 4, 1300, 120, True, 0.25, (1, True)),
]


@pytest.mark.parametrize("B,l_x,H,s0,l_s,causal,p_drop,form", FORWARD)
def test_forward_of_four_groups_against_the_oracle(B, l_x, H, s0, l_s, causal, p_drop, form):
    plan = fwd_plan(B, l_x, H, 64, s0, l_s, causal, p_drop > 0)
    assert (plan.row_blocks, plan.groups, plan.splits > 1) == form
    Q, K, V, _ = stage_all(B, l_x, H, 64, 9500 + l_x, "bf16")
    sl, heads = slice(s0, s0 + l_s), slice(0, 2 if B == 1 else H)      # (one batch's heads do not depend on each other: two are enough)
    drop = {"p_drop": p_drop, "seed": 77} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(Q.dev[:, sl].contiguous(), K.dev, V.dev, s0, causal, **drop)
    args = (Q.f64[:, sl, heads], K.f64[:, :, heads], V.f64[:, :, heads], s0, causal)
    ref, ref_lse = oracle.segment_fwd_dropout(*args, p_drop, 77) if p_drop else oracle.segment_fwd(*args)
    assert rel_err(to_np(out)[:, :, heads], ref) <= TOL["bf16"]["t"]
    assert lse_err(to_np(lse)[:, heads], ref_lse) <= TOL["bf16"]["lse"]


@pytest.mark.parametrize("B,l_x,H,s0,l_s,causal,p_drop,form", BACKWARD)
def test_backward_of_narrow_wavefronts_against_the_oracle(B, l_x, H, s0, l_s, causal, p_drop, form):
    plan = bwd_plan(B, l_x, H, 64, s0, l_s, causal, p_drop > 0)
    assert plan.narrow and not plan.one_pass and (plan.own, plan.splits > 1) == form
    Q, K, V, DO = stage_all(B, l_x, H, 64, 9600 + l_x, "bf16")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    drop = {"p_drop": p_drop, "seed": 78} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, causal, **drop)
    args = (Q.f64[:, sl], K.f64, V.f64, DO.f64[:, sl], s0, causal)
    ref = oracle.segment_bwd_dropout(*args, p_drop, 78) if p_drop else oracle.segment_bwd(*args)
    grads = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    over = out.clone()                                  # a gradient written over the forward's output: D from a launch of its own
    for got in (grads, lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, over, lse, do, causal, dq=over, **drop)):
        for name, g, want in zip(("dq", "dk", "dv"), got, ref):
            assert rel_err(to_np(g), want) <= TOL["bf16"]["t"], name
    again = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal, **drop)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))

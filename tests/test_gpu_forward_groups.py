"""Forward workgroups whose wavefronts form two groups with a part of the keys each: sizes at which the second group has
no key tile, one, a partial one, or one less than the first, and at which rows of the last query tile do not exist."""
import pytest

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, fwd_plan, lse_err, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, d, s0, l_s, causal
    (1, 1, 1, 64, 0, 1, True), (2, 64, 3, 64, 0, 64, True), (1, 65, 2, 64, 0, 65, False), (2, 190, 2, 64, 100, 33, True),
    (3, 257, 2, 64, 192, 65, True), (1, 320, 5, 64, 0, 320, True), (2, 448, 2, 64, 3, 97, False), (4, 700, 4, 64, 611, 70, True),
    (2, 900, 9, 64, 200, 700, True),
    (1, 1, 1, 128, 0, 1, False), (2, 65, 2, 128, 1, 33, True), (1, 129, 3, 128, 0, 129, True), (4, 330, 4, 128, 200, 130, False),
    (2, 1100, 8, 128, 100, 1000, True),
]


# The workgroup's form by row blocks of 32 x groups, and whether the keys are split besides: every one that is built, with
# rows past the end in the last query tile.  (At d = 64 and with dropout there is no 4 x 2.)
FORMS = [  # B, l_x, H, d, s0, l_s, causal, p_drop, (row blocks, groups, split)
    (1, 200, 1, 64, 0, 125, True, 0.0, (2, 2, False)), (1, 718, 1, 64, 602, 85, False, 0.0, (2, 2, True)),
    (1, 546, 64, 64, 0, 546, True, 0.0, (4, 1, False)), (1, 3395, 24, 64, 2620, 686, False, 0.0, (4, 1, True)),
    (1, 710, 24, 64, 0, 710, False, 0.0, (4, 2, False)), (1, 2609, 16, 64, 1648, 598, False, 0.0, (4, 2, True)),
    (1, 195, 1, 64, 102, 73, True, 0.25, (2, 2, False)), (1, 807, 1, 64, 610, 70, True, 0.25, (2, 2, True)),
    (1, 695, 64, 64, 0, 695, False, 0.25, (4, 1, False)), (1, 1996, 16, 64, 0, 1185, False, 0.25, (4, 1, True)),
    (1, 206, 1, 128, 0, 206, True, 0.0, (4, 2, False)), (1, 642, 1, 128, 414, 209, False, 0.0, (4, 2, True)),
    (1, 691, 48, 128, 0, 691, False, 0.0, (8, 1, False)), (1, 1187, 1, 128, 190, 413, True, 0.0, (8, 1, True)),
    (1, 181, 1, 128, 0, 181, True, 0.25, (4, 2, False)), (1, 514, 1, 128, 182, 303, False, 0.25, (4, 2, True)),
    (1, 700, 48, 128, 0, 700, False, 0.25, (8, 1, False)), (1, 2203, 24, 128, 1052, 706, False, 0.25, (8, 1, True)),
]


def check(B, l_x, H, d, s0, l_s, causal, p_drop, seed):
    Q, K, V, _ = stage_all(B, l_x, H, d, seed, "bf16")
    sl, heads = slice(s0, s0 + l_s), slice(0, 2 if B == 1 else H)      # (one batch's heads do not depend on each other: two are enough)
    drop = {"p_drop": p_drop, "seed": 77} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(Q.dev[:, sl].contiguous(), K.dev, V.dev, s0, causal, **drop)
    args = (Q.f64[:, sl, heads], K.f64[:, :, heads], V.f64[:, :, heads], s0, causal)
    ref, ref_lse = oracle.segment_fwd_dropout(*args, p_drop, 77) if p_drop else oracle.segment_fwd(*args)
    assert rel_err(to_np(out)[:, :, heads], ref) <= TOL["bf16"]["t"]
    assert lse_err(to_np(lse)[:, heads], ref_lse) <= TOL["bf16"]["lse"]


@pytest.mark.parametrize("p_drop", [0.0, 0.25])
@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal", SHAPES)
def test_forward_against_the_oracle(B, l_x, H, d, s0, l_s, causal, p_drop):
    check(B, l_x, H, d, s0, l_s, causal, p_drop, 9300 + l_x + d)


@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal,p_drop,form", FORMS)
def test_every_form_against_the_oracle(B, l_x, H, d, s0, l_s, causal, p_drop, form):
    plan = fwd_plan(B, l_x, H, d, s0, l_s, causal, p_drop > 0)
    assert (plan.row_blocks, plan.groups, plan.splits > 1) == form
    check(B, l_x, H, d, s0, l_s, causal, p_drop, 9350 + l_x + d)

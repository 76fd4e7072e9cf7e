"""Forward workgroups whose wavefronts form two groups with a part of the keys each: sizes at which the second group has
no key tile, one, a partial one, or one less than the first, and at which rows of the last query tile do not exist."""
import pytest

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, lse_err, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, d, s0, l_s, causal
    (1, 1, 1, 64, 0, 1, True), (2, 64, 3, 64, 0, 64, True), (1, 65, 2, 64, 0, 65, False), (2, 190, 2, 64, 100, 33, True),
    (3, 257, 2, 64, 192, 65, True), (1, 320, 5, 64, 0, 320, True), (2, 448, 2, 64, 3, 97, False), (4, 700, 4, 64, 611, 70, True),
    (2, 900, 9, 64, 200, 700, True),                                                     # 64-row and 128-row tiles, both in groups
    (1, 1, 1, 128, 0, 1, False), (2, 65, 2, 128, 1, 33, True), (1, 129, 3, 128, 0, 129, True), (4, 330, 4, 128, 200, 130, False),
    (2, 1100, 8, 128, 100, 1000, True),
]


@pytest.mark.parametrize("p_drop", [0.0, 0.25])
@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal", SHAPES)
def test_forward_against_the_oracle(B, l_x, H, d, s0, l_s, causal, p_drop):
    Q, K, V, _ = stage_all(B, l_x, H, d, 9300 + l_x + d, "bf16")
    sl = slice(s0, s0 + l_s)
    drop = {"p_drop": p_drop, "seed": 77} if p_drop else {}
    out, lse = lss.lss_segment_attn_fwd(Q.dev[:, sl].contiguous(), K.dev, V.dev, s0, causal, **drop)
    if p_drop:
        ref, ref_lse = oracle.segment_fwd_dropout(Q.f64[:, sl], K.f64, V.f64, s0, causal, p_drop, 77)
    else:
        ref, ref_lse = oracle.segment_fwd(Q.f64[:, sl], K.f64, V.f64, s0, causal)
    assert rel_err(to_np(out), ref) <= TOL["bf16"]["t"]
    assert lse_err(to_np(lse), ref_lse) <= TOL["bf16"]["lse"]

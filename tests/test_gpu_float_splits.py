"""Single precision: launches whose keys are split over several dQ workgroups because the chip is idle otherwise, at sizes where a range
is partial, a wavefront has rows of one 16-row block only, or the last ranges see no key; and the forward's maximum
raised late: rows whose scores grow along the keys."""
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss
from _util import TOL, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, d, s0, l_s, causal
    (1, 1000, 2, 64, 0, 100, False), (1, 1000, 2, 64, 900, 100, True), (1, 2000, 1, 64, 100, 17, True), (2, 700, 1, 64, 200, 33, True),
    (1, 1500, 2, 64, 1100, 400, True), (1, 1000, 2, 128, 500, 300, True), (1, 1300, 1, 128, 17, 15, True), (1, 521, 2, 128, 0, 130, False),
]


@pytest.mark.parametrize("growth", [0.0, 40.0])
@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal", SHAPES)
def test_against_the_oracle(B, l_x, H, d, s0, l_s, causal, growth):
    Q, K, V, DO = stage_all(B, l_x, H, d, 5100 + l_x + l_s, "f32")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    q[..., 0] = 1.0
    k = K.dev.clone()
    k[..., 0] += growth * torch.arange(l_x, device=k.device)[None, :, None] / l_x       # scores rise by growth / sqrt(d)
    q64, k64 = to_np(q).astype("float64"), to_np(k).astype("float64")
    out, lse = lss.lss_segment_attn_fwd(q, k, V.dev, s0, causal)
    grads = lss.lss_segment_attn_bwd(q, k, V.dev, s0, out, lse, do, causal)
    ref_out, ref_lse = oracle.segment_fwd(q64, k64, V.f64, s0, causal)
    ref = oracle.segment_bwd(q64, k64, V.f64, DO.f64[:, sl], s0, causal)
    for name, got, want in zip(("out", "dq", "dk", "dv"), (out, *grads), (ref_out, *ref)):
        assert rel_err(to_np(got), want) <= TOL["f32"]["t"], name
    assert abs(to_np(lse) - ref_lse).max() <= TOL["f32"]["lse"]
    again = lss.lss_segment_attn_bwd(q, k, V.dev, s0, out, lse, do, causal)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))

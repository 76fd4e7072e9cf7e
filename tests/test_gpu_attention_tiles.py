"""Attention launches on either side of the choices the launchers make by size (two wavefronts per key block or one,
how many key splits, which XCD gets which head), at ragged row and key counts, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss, timing
from _util import rel_err, stage_all, to_np
from test_gpu_parity import run_segment

pytestmark = pytest.mark.gpu

SHAPES = [  # B, l_x, H, d, s0, l_s, causal
    (1, 129, 1, 64, 64, 65, True),          # one key past a tile of 128, one row past a tile of 64
    (2, 700, 3, 64, 333, 97, True), (2, 700, 3, 128, 333, 97, True),
    (1, 1100, 2, 64, 33, 1029, True), (1, 1100, 2, 64, 0, 1029, False),
    (2, 900, 50, 64, 700, 130, True),       # 800 key tiles: one wavefront per key block
    (1, 2500, 2, 128, 1000, 70, False),
    (3, 260, 11, 64, 0, 260, True), (1, 2000, 13, 64, 1700, 300, True),     # heads that the eight XCDs share
    (2, 1500, 27, 64, 1200, 65, True), (1, 700, 9, 128, 5, 300, False),
    (1, 2752, 2, 64, 2240, 512, True), (1, 2752, 2, 64, 2239, 513, True),   # the backward's row sums: within its workgroups or ahead
    # few rows, many keys: all gradients in one pass, with two, three and four blocks of 32 rows
    (1, 1403, 20, 64, 1203, 58, True), (1, 1403, 20, 64, 900, 33, False), (3, 1500, 11, 64, 1436, 64, True), (1, 1440, 24, 64, 7, 1, False),
    (2, 1480, 20, 64, 1350, 65, True), (2, 1480, 20, 64, 100, 96, False), (2, 2001, 32, 64, 1830, 128, True), (2, 1990, 32, 64, 1500, 97, False),
]


@pytest.mark.parametrize("kind", ["bf16", "f32"])
@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal", SHAPES)
def test_matches_oracle(B, l_x, H, d, s0, l_s, causal, kind):
    Q, K, V, DO = stage_all(B, l_x, H, d, 8800 + l_x + H, kind)
    run_segment(Q, K, V, DO, s0, l_s, causal, kind, tag=f"{(B, l_x, H, d, s0, l_s, causal, kind)}")


@pytest.mark.parametrize("d", [64, 128])
def test_float_results_are_those_of_single_precision(d):
    # three bf16 parts per float: errors of a few units in the last place, not of a bf16 product
    B, l_x, H, s0, l_s = 1, 800, 2, 250, 300
    Q, K, V, DO = stage_all(B, l_x, H, d, 8900 + d, "f32", std=2.0)
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, True)
    dq, dk, dv = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, True)
    ro, rl = oracle.segment_fwd(Q.f64[:, sl], K.f64, V.f64, s0, True)
    ref = (ro, rl, *oracle.segment_bwd(Q.f64[:, sl], K.f64, V.f64, DO.f64[:, sl], s0, True))
    for name, got, want in zip(("out", "lse", "dq", "dk", "dv"), (out, lse, dq, dk, dv), ref):
        assert rel_err(to_np(got), want) <= 1e-5, name
    again = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, True)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again))


@pytest.mark.parametrize("B,l_x,H,d,s0,l_s,causal", [(1, 1024, 4, 64, 256, 256, True), (1, 1024, 4, 64, 768, 256, True), (1, 2000, 4, 64, 1900, 58, True),
                                                     (1, 1500, 8, 128, 100, 130, False)])
def test_split_forward_rounds_its_output_once(B, l_x, H, d, s0, l_s, causal):
    # Launches of few query tiles split the keys and merge.  Rounding a Gaussian value to bf16 costs 1.65e-3 of its size
    # (root mean square).  A row's weights are rounded as matrix operands, its result at the end: 1.65e-3 * sqrt(2) = 2.33e-3.
    # Partial results that were rounded to bf16 on their way to the merge would make it sqrt(3), 2.86e-3; the line lies at sqrt(2.4).
    Q, K, V, _ = stage_all(B, l_x, H, d, 8950 + l_s, "bf16")
    sl = slice(s0, s0 + l_s)
    merge = {n: i for i, n in timing.kernel_names().items()}["fwd_merge_kernel"]
    timing.reset()
    timing.enable(True)
    try:
        out, _ = lss.lss_segment_attn_fwd(Q.dev[:, sl].contiguous(), K.dev, V.dev, s0, causal)
        assert timing.read(merge)[1] == 1
    finally:
        timing.enable(False)
    ref, _ = oracle.segment_fwd(Q.f64[:, sl], K.f64, V.f64, s0, causal)
    assert np.linalg.norm(to_np(out) - ref) <= 2.55e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("d,causal", [(64, True), (64, False), (128, True)])
def test_float_errors_are_no_larger_than_stated(d, causal):
    # Figures of lss_f32.hip (2-norm of the difference over 2-norm of the result) and a fifth more, for other inputs and orders
    # of the sums.  What they tell apart: products of two parts per float are off by 2^-17 and more, 4e-6; gradients of
    # the queries added up product by product 6.6e-7.
    B, l_x, H, s0, l_s = 1, 2000, 2, 1488 if causal else 700, 512
    Q, K, V, DO = stage_all(B, l_x, H, d, 8970 + d, "f32")
    sl = slice(s0, s0 + l_s)
    q, do = Q.dev[:, sl].contiguous(), DO.dev[:, sl].contiguous()
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, causal)
    grads = lss.lss_segment_attn_bwd(q, K.dev, V.dev, s0, out, lse, do, causal)
    ro, _ = oracle.segment_fwd(Q.f64[:, sl], K.f64, V.f64, s0, causal)
    ref = oracle.segment_bwd(Q.f64[:, sl], K.f64, V.f64, DO.f64[:, sl], s0, causal)
    for name, got, want, most in zip(("out", "dq", "dk", "dv"), (out, *grads), (ro, *ref), (5.7e-7, 6.2e-7, 7.3e-7, 7.4e-7)):
        err = np.linalg.norm(to_np(got) - want) / np.linalg.norm(want)
        assert err <= most, (name, err)

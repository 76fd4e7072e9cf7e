"""Single precision over the whole range of float: what the three bf16 parts of a value miss -- infinities, NaNs, values whose
first part overflows, values so small that the last part is subnormal -- gives the results of fp32 arithmetic all the same."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss, synth
from _util import Staged, to_np

pytestmark = pytest.mark.gpu

# B, l_x, H, d, s0, l_s, causal: key blocks shared by two wavefronts (few heads) and held by one, split keys, both widths
SHAPES = [(1, 300, 1, 64, 150, 100, True), (1, 300, 1, 64, 150, 100, False), (2, 900, 50, 64, 700, 130, True), (1, 2000, 2, 64, 1500, 58, True),
          (1, 300, 2, 128, 150, 100, True), (1, 700, 2, 128, 100, 200, False)]
# Errors (2-norm) of these shapes in range: at most 7e-7.  Beyond it fp32 products give the same and subnormal results a little more.
MOST = 1e-6


def _inputs(B, l_x, H, d, s0, l_s, seed=77):
    q, k, v, do = synth.make_inputs(B, l_x, H, d, seed, 1.0)
    return q[:, s0:s0 + l_s].copy(), k, v, do[:, s0:s0 + l_s].copy()


def _run(q, k, v, do, s0, causal, **drop):
    Q, K, V, G = (Staged(a, "f32") for a in (q, k, v, do))
    out, lse = lss.lss_segment_attn_fwd(Q.dev, K.dev, V.dev, s0, causal, **drop)
    return (out, lse, *lss.lss_segment_attn_bwd(Q.dev, K.dev, V.dev, s0, out, lse, G.dev, causal, **drop))


def _check(q, k, v, do, s0, causal):
    got = _run(q, k, v, do, s0, causal)
    q, k, v, do = (a.astype(np.float64) for a in (q, k, v, do))
    ref = (oracle.segment_fwd(q, k, v, s0, causal)[0], None, *oracle.segment_bwd(q, k, v, do, s0, causal))
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), got, ref):
        if b is None:
            continue
        a = to_np(a)
        assert np.isfinite(a).all(), name
        size = np.abs(b).max()          # (squares of numbers this small or large would leave the range of float64's own exponents)
        err = np.linalg.norm((a - b) / size) / np.linalg.norm(b / size)
        assert err <= MOST, (name, err)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("which", ["v", "do", "k and q", "q and k", "part of v"])
def test_tiny_values(shape, which):
    B, l_x, H, d, s0, l_s, causal = shape
    q, k, v, do = _inputs(*shape[:6])
    t = np.float32(2.0 ** -113)         # three parts hold 13 of its 24 bits
    if which == "v":
        v *= t
    elif which == "do":
        do *= t
    elif which == "k and q":            # the scores stay as they are
        k *= t; q /= t
    elif which == "q and k":
        q *= t; k /= t
    else:                               # tiny values, zeros and ordinary ones side by side
        v[:, :, :, : d // 4] *= t
        v[:, :, :, d // 4: d // 2] = 0.0
    _check(q, k, v, do, s0, causal)


@pytest.mark.parametrize("shape", SHAPES)
def test_zeros_are_ordinary_values(shape):
    q, k, v, do = _inputs(*shape[:6])
    for a in (q, k, v, do):
        a[..., 1::2] = 0.0
    do[:, ::3] = 0.0
    _check(q, k, v, do, shape[4], shape[6])


@pytest.mark.parametrize("shape", SHAPES)
def test_values_whose_first_part_overflows(shape):
    B, l_x, H, d, s0, l_s, causal = shape
    q, k, v, do = _inputs(*shape[:6])
    k[0, 37, 0, 5] = -3.4e38            # bf16 ends at 3.39e38
    q[..., 5] *= 1e-38
    _check(q, k, v, do, s0, causal)
    q, k, v, do = _inputs(*shape[:6])
    v[0, 37, 0, 5] = 3.4e38
    Q, K, V, _ = (Staged(a, "f32") for a in (q, k, v, do))
    out, _ = lss.lss_segment_attn_fwd(Q.dev, K.dev, V.dev, s0, causal)
    ref, _ = oracle.segment_fwd(Q.f64, K.f64, V.f64, s0, causal)
    assert (np.abs(to_np(out) - ref) <= 1e-5 * np.abs(ref) + 1e-5).all()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_infinite_and_nan_values(shape, value):
    B, l_x, H, d, s0, l_s, causal = shape
    q, k, v, do = _inputs(*shape[:6])
    key = s0 + l_s // 2
    v[0, key, 0, 5] = value
    Q, K, V = (Staged(a, "f32") for a in (q, k, v))
    out = to_np(lss.lss_segment_attn_fwd(Q.dev, K.dev, V.dev, s0, causal)[0])
    first = l_s // 2 if causal else 0   # rows from here on see the key with a weight above 0
    hit = out[0, first:, 0, 5]
    assert np.isnan(hit).all() if np.isnan(value) else (hit == value).all()
    out[0, :, 0, 5] = 0.0
    assert np.isfinite(out).all()       # other columns, heads and batch entries
    # rows of other wavefronts' blocks that do not see the key
    if causal and l_s // 2 >= 64:
        again = to_np(lss.lss_segment_attn_fwd(Q.dev, K.dev, V.dev, s0, causal)[0])
        assert np.isfinite(again[0, : l_s // 2 - 63, 0, 5]).all()


@pytest.mark.parametrize("value", [float("inf"), 3.4e38])
def test_infinite_gradients_reach_the_right_keys(value):
    # dO infinite in one row and column: dV of the keys that row sees is infinite in that column, everything else of dV finite
    s0, l_s, d = 150, 100, 64
    q, k, v, do = _inputs(1, 300, 1, d, s0, l_s)
    do[0, 7, 0, 5] = value
    dv = to_np(_run(q, k, v, do, s0, False)[4])
    col = dv[0, :, 0, 5].copy()
    assert (col == value).all() if np.isinf(value) else np.isfinite(col).all()
    dv[0, :, 0, 5] = 0.0
    assert np.isfinite(dv).all()


@pytest.mark.parametrize("d", [64, 128])
def test_dropout_gradients_scale_with_theirs(d):
    # the gradients are linear in dO: 2^-113 dO gives 2^-113 times the gradients, with the same decisions
    s0, l_s = 150, 100
    q, k, v, do = _inputs(1, 300, 2, d, s0, l_s)
    drop = dict(p_drop=0.2, seed=11)
    t = np.float32(2.0 ** -113)
    for a, b in zip(_run(q, k, v, do, s0, True, **drop)[2:], _run(q, k, v, do * t, s0, True, **drop)[2:]):
        a, b = to_np(a), to_np(b) / float(t)
        assert np.linalg.norm(a - b) <= MOST * np.linalg.norm(a)
    vt = v * t
    a, b = to_np(_run(q, k, v, do, s0, True, **drop)[0]), to_np(_run(q, k, vt, do, s0, True, **drop)[0]) / float(t)
    assert np.linalg.norm(a - b) <= MOST * np.linalg.norm(a)

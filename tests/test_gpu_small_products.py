"""Products of few rows or columns: tiles of 32 x 64 and 32 x 32 whose groups of wavefronts share the contraction, and 128 x 128 tiles of eight
wavefronts with four contraction tiles on their way.  Remainders in rows, columns that end inside a block of tiles, contractions shorter than
the number of groups, and rows that do not fill a contraction tile (weight gradient)."""
import pytest
import torch

from paper_2311_02382_amd import lss, synth
from _util import Staged, TOL, rel_err, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, K, N
    (1, 256, 640), (31, 512, 128), (33, 1152, 384), (58, 4096, 256), (97, 128, 1024), (200, 384, 1536),     # 32 rows, 64 or 32 columns
    (63, 640, 640), (450, 512, 512), (600, 1024, 256),                                                      # weight gradients in them too
    (2047, 512, 2048), (1921, 640, 1920),                                                                   # 128 x 128, one per compute unit
]


def _staged(seed, shape, std=1.0):
    n = 1
    for x in shape:
        n *= x
    return Staged(synth.normal_f32(seed, n, std).reshape(shape), "bf16")


@pytest.mark.parametrize("rows,K,N", SHAPES)
def test_linear_maps_and_weight_gradient(rows, K, N):
    A, W, DC = _staged(9700 + rows, (rows, K)), _staged(9701 + rows, (K, N), K ** -0.5), _staged(9702 + rows, (rows, N))
    t = TOL["bf16"]["t"]
    c = lss.lss_linear_fwd(A.dev, W.dev)
    assert rel_err(to_np(c), A.f64 @ W.f64) <= t
    u, g = lss.lss_linear_gelu_fwd(A.dev, W.dev)
    assert torch.equal(u, c) and torch.equal(g, lss.lss_gelu_fwd(c))
    da = lss.lss_linear_bwd_input(DC.dev, W.dev)
    assert rel_err(to_np(da), DC.f64 @ W.f64.T) <= t
    assert torch.equal(lss.lss_linear_bwd_input_gelu(DC.dev, W.dev, A.dev), lss.lss_gelu_bwd(A.dev, da))
    dw = lss.lss_linear_bwd_weight(A.dev, DC.dev)
    assert rel_err(to_np(dw), A.f64.T @ DC.f64) <= TOL["f32"]["t"]
    assert torch.equal(dw, lss.lss_linear_bwd_weight(A.dev, DC.dev))


@pytest.mark.parametrize("B,l_x,H,s0,l_s", [(1, 512, 2, 256, 127), (1, 601, 4, 100, 300), (2, 90, 6, 30, 41), (1, 1024, 8, 512, 256), (1, 2000, 4, 300, 57)])
def test_projections_in_small_tiles(B, l_x, H, s0, l_s):
    d, E, rv = 64, 64 * H, s0 + l_s
    X, WQ, WKV = _staged(9800 + l_x, (B, l_x, E)), _staged(9801 + l_x, (E, E), E ** -0.5), _staged(9802 + l_x, (E, 2 * E), E ** -0.5)
    q, k, v = lss.lss_project_qkv(X.dev, WQ.dev, WKV.dev, s0, l_s, H)
    t = TOL["bf16"]["t"]
    assert rel_err(to_np(q.view(B, l_s, E)), X.f64[:, s0:rv] @ WQ.f64) <= t
    kv = X.f64 @ WKV.f64
    assert rel_err(to_np(k.view(B, l_x, E)), kv[..., :E]) <= t and rel_err(to_np(v.view(B, l_x, E)), kv[..., E:]) <= t
    dk, dv = (Staged(synth.normal_f32(9803 + i + l_x, B * l_x * E, 1.0).reshape(B, l_x, H, d), "f32") for i in range(2))
    dk.dev[:, rv:] = float("nan")       # rows past rows_valid are never read
    dv.dev[:, rv:] = float("nan")
    DQ = _staged(9805 + l_x, (B, l_s, H, d))
    dx_q, dx = lss.lss_project_bwd(DQ.dev, dk.dev, dv.dev, WQ.dev, WKV.dev, rv)
    assert rel_err(to_np(dx_q), DQ.f64.reshape(B, l_s, E) @ WQ.f64.T) <= t
    dkf, dvf = dk.f64.reshape(B, l_x, E)[:, :rv], dv.f64.reshape(B, l_x, E)[:, :rv]
    assert rel_err(to_np(dx[:, :rv]), dkf @ WKV.f64[:, :E].T + dvf @ WKV.f64[:, E:].T) <= t
    assert not dx[:, rv:].any()
    dwq, dwkv = lss.lss_project_bwd_weight(X.dev, DQ.dev, dk.dev, dv.dev, s0, rv)
    rows = X.f64[:, :rv].reshape(-1, E)
    assert rel_err(to_np(dwkv[:, :E]), rows.T @ dkf.reshape(-1, E)) <= t
    assert rel_err(to_np(dwkv[:, E:]), rows.T @ dvf.reshape(-1, E)) <= t
    assert rel_err(to_np(dwq), X.f64[:, s0:rv].reshape(-1, E).T @ DQ.f64.reshape(-1, E)) <= t

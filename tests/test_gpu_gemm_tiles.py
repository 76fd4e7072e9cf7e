"""The GEMM's tile sizes: a launch takes 256-, 128- or 64-wide tiles, with or without wavefront groups that share the
contraction, by its size.  Sizes here have remainders in rows, a contraction shorter than the number of groups, and rows that
do not fill a contraction tile (weight gradient).  (test_gpu_product_tiles.py names the tile of every size.)"""
import pytest
import torch

from paper_2311_02382_amd import lss, synth
from _util import Staged, TOL, rel_err, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, K, N
    (1, 128, 128), (33, 128, 1024), (65, 2048, 128), (129, 4096, 256),      # 64 x 64 and 32 x 32 tiles, whose groups share long contractions
    (700, 1024, 1024), (2049, 512, 512),                                    # 64 x 64, about one workgroup per compute unit
    (1300, 640, 2560), (4100, 1280, 640),                                   # 128 x 128 in one direction
    (8200, 1024, 2048),                                                     # 128 x 128 in all
]


def _staged(seed, shape, std=1.0):
    n = 1
    for x in shape:
        n *= x
    return Staged(synth.normal_f32(seed, n, std).reshape(shape), "bf16")


@pytest.mark.parametrize("rows,K,N", SHAPES)
def test_linear_maps_and_weight_gradient(rows, K, N):
    A, W, DC = _staged(9100 + rows, (rows, K)), _staged(9101 + rows, (K, N), K ** -0.5), _staged(9102 + rows, (rows, N))
    t = TOL["bf16"]["t"]
    assert rel_err(to_np(lss.lss_linear_fwd(A.dev, W.dev)), A.f64 @ W.f64) <= t
    assert rel_err(to_np(lss.lss_linear_bwd_input(DC.dev, W.dev)), DC.f64 @ W.f64.T) <= t
    dw = lss.lss_linear_bwd_weight(A.dev, DC.dev)
    assert rel_err(to_np(dw), A.f64.T @ DC.f64) <= TOL["f32"]["t"]
    assert torch.equal(dw, lss.lss_linear_bwd_weight(A.dev, DC.dev))


@pytest.mark.parametrize("B,l_x,H,s0,l_s", [(1, 70, 2, 3, 66), (3, 1000, 4, 437, 300), (2, 4100, 8, 2000, 1044)])
def test_projections_across_tile_sizes(B, l_x, H, s0, l_s):
    d, E, rv = 64, 64 * H, s0 + l_s
    X, WQ, WKV = _staged(9200 + l_x, (B, l_x, E)), _staged(9201 + l_x, (E, E), E ** -0.5), _staged(9202 + l_x, (E, 2 * E), E ** -0.5)
    q, k, v = lss.lss_project_qkv(X.dev, WQ.dev, WKV.dev, s0, l_s, H)
    t = TOL["bf16"]["t"]
    assert rel_err(to_np(q.view(B, l_s, E)), X.f64[:, s0:rv] @ WQ.f64) <= t
    kv = X.f64 @ WKV.f64
    assert rel_err(to_np(k.view(B, l_x, E)), kv[..., :E]) <= t and rel_err(to_np(v.view(B, l_x, E)), kv[..., E:]) <= t
    # float partials, rows past rows_valid never read
    dk, dv = (Staged(synth.normal_f32(9203 + i + l_x, B * l_x * E, 1.0).reshape(B, l_x, H, d), "f32") for i in range(2))
    dk.dev[:, rv:] = float("nan")
    dv.dev[:, rv:] = float("nan")
    DQ = _staged(9205 + l_x, (B, l_s, H, d))
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

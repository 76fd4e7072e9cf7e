"""Products of few rows or columns: tiles of 32 x 64 and 32 x 32 whose groups of wavefronts share the contraction, and 128 x 128 tiles of eight
wavefronts with four contraction tiles on their way.  Remainders in rows, columns that end inside a block of tiles, contractions shorter than
the number of groups, and rows that do not fill a contraction tile (weight gradient).  (test_gpu_product_tiles.py names the tile of every size.)"""
import pytest
import torch

from paper_2311_02382_amd import lss, synth
from _util import Staged, TOL, project_plan, rel_err, to_np

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, K, N
    (1, 256, 640), (31, 512, 128), (33, 1152, 384), (58, 4096, 256), (97, 128, 1024), (200, 384, 1536),     # 32 rows, 64 or 32 columns
    (63, 640, 640), (450, 512, 512), (600, 1024, 256),                                                      # the last two's weight gradients in them too
    (2047, 512, 2048), (1921, 640, 1920),                                                                   # forward in 128 x 128, one per compute unit
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


@pytest.mark.parametrize("skip_tail", [False, True])
@pytest.mark.parametrize("tile,B,l_x,H,l_s,rows_valid", [
    ("32x32", 1, 340, 2, 22, 24), ("32x32", 3, 700, 2, 32, 32), ("32x64", 1, 1280, 2, 89, 931), ("64x64 in groups", 1, 612, 14, 14, 292),
    ("64x64", 2, 2276, 2, 98, 1946), ("128x128 by two", 1, 2303, 16, 88, 1988), ("128x128", 2, 2449, 16, 117, 2124), ("256x256", 1, 17000, 8, 200, 16500),
])
def test_rows_without_data_are_cleared(tile, B, l_x, H, l_s, rows_valid, skip_tail):
    """project_bwd clears them 64 KB at a time, or a tile where that is more: to the last row and no further, and with skip_masked_tail to the next multiple of 256."""
    d, E = 64, 64 * H
    assert project_plan(1, B, l_x, H, d, l_s, rows_valid) == tile
    gen = torch.Generator(device="cuda").manual_seed(l_x + rows_valid)
    WQ, WKV, DQ = ((torch.randn(shape, generator=gen, device="cuda") * std).to(torch.bfloat16)
                   for shape, std in (((E, E), E ** -0.5), ((E, 2 * E), E ** -0.5), ((B, l_s, H, d), 1.0)))
    dk, dv = (torch.randn((B, l_x, H, d), generator=gen, device="cuda") for _ in range(2))
    dk[:, rows_valid:] = float("nan")
    dv[:, rows_valid:] = float("nan")
    canary = -7.25
    room = torch.full((B * l_x + 512, E), canary, device="cuda")
    dx_q, dx = lss.lss_project_bwd(DQ, dk, dv, WQ, WKV, rows_valid, dx_partial=room[:B * l_x].view(B, l_x, E), skip_masked_tail=skip_tail)
    end = min(l_x, -(-rows_valid // 256) * 256) if skip_tail else l_x
    assert not dx[:, rows_valid:end].any() and (dx[:, end:] == canary).all() and (room[B * l_x:] == canary).all()
    W = WKV.double()
    for b in range(B):
        rows = torch.cat([t[b, :rows_valid].reshape(-1, E).to(torch.bfloat16).double() for t in (dk, dv)], 1)
        want = rows @ torch.cat([W[:, :E], W[:, E:]], 1).T
        assert (dx[b, :rows_valid].double() - want).abs().max() <= TOL["f32"]["t"] * want.abs().max()
        want = DQ[b].reshape(-1, E).double() @ WQ.double().T
        assert (dx_q[b].double() - want).abs().max() <= TOL["f32"]["t"] * want.abs().max()

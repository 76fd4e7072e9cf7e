"""Every tile that a matrix product has a kernel for, in every product that takes it, against 64-bit products of the same operands.  The tile that a size
takes is asked of the library (csrc/lss_plan.h), so that a change to the rule shows which sizes have left theirs.  Rows and columns end inside a
tile wherever there is such a size.  Contractions longer than what is on its way at once, shared by groups of wavefronts unevenly, are those of the larger tiles
everywhere, and of the 32-wide ones in ROUNDS below."""
import pytest
import torch

from paper_2311_02382_amd import lss
from _util import TOL, linear_form, linear_plan, project_form, project_plan

LINEAR = {  # tile: rows, K, N  (contraction over K)
    "fwd": {"32x32": (45, 1152, 384), "32x64": (58, 512, 4480), "64x64": (70, 512, 5504), "64x64 in groups": (67, 768, 6016),
            "128x128 of eight": (1925, 640, 1920), "128x128": (658, 512, 5760), "256x256": (2224, 512, 5504)},
    # (contraction over N)
    "bwd_input": {"32x32": (45, 384, 1152), "32x64": (58, 4224, 512), "64x64": (66, 5760, 512), "64x64 in groups": (70, 5504, 768),
                  "128x128 of eight": (1925, 1920, 640), "128x128": (772, 4736, 512), "256x256": (2698, 4480, 512)},
}
LINEAR["fwd"]["128x128 of eight, whole rows"], LINEAR["bwd_input"]["128x128 of eight, whole rows"] = (2048, 512, 2048), (2048, 2048, 512)
WEIGHT = {  # (tile, rows in chunks): rows, K, N  (contraction over the rows)
    ("32x32", False): (450, 128, 256), ("32x32", True): (2567, 128, 128), ("32x64", False): (450, 384, 384), ("32x64", True): (6161, 128, 128),
    ("64x64", False): (515, 640, 1664), ("64x64", True): (2571, 128, 1152), ("64x64 in groups", False): (517, 384, 1408),
    ("64x64 in groups", True): (3077, 384, 384), ("128x128 by two", False): (533, 384, 5504), ("128x128 by two", True): (6277, 128, 2176),
    ("128x128", False): (517, 4736, 896), ("128x128", True): (3411, 384, 3712), ("256x256", False): (515, 1664, 5248), ("256x256", True): (2507, 4736, 896),
}
PROJECT = {  # B, l_x, H, l_s, rows_valid
    "qkv": {"32x32": (1, 125, 6, 49, 115), "32x64": (1, 135, 4, 75, 81), "64x64": (2, 342, 4, 323, 338), "64x64 in groups": (1, 228, 12, 187, 195),
            "128x128 of eight": (2, 1429, 4, 1244, 1322), "128x128": (3, 2001, 4, 1368, 1422), "256x256": (3, 7527, 4, 1421, 5412)},
    "bwd": {"32x32": (1, 135, 4, 75, 81), "32x64": (2, 142, 4, 108, 132), "64x64": (3, 376, 4, 329, 373), "64x64 in groups": (2, 765, 4, 299, 747),
            "128x128 by two": (3, 1569, 4, 1305, 1552), "128x128": (3, 2341, 6, 1415, 2279), "256x256": (3, 7967, 6, 1476, 7384)},
}
PARTIALS = {  # (tile of dW_kv, rows in chunks): B, l_x, H, l_s, rows_valid
    ("32x32", False): (1, 206, 4, 100, 204), ("64x64", False): (1, 135, 4, 75, 81), ("64x64", True): (3, 535, 4, 286, 531),
    ("64x64 in groups", False): (2, 267, 4, 148, 261), ("64x64 in groups", True): (2, 519, 4, 429, 514), ("128x128 by two", False): (2, 269, 12, 163, 266),
    ("128x128 by two", True): (3, 971, 8, 873, 971), ("128x128", False): (2, 135, 12, 43, 76), ("128x128", True): (2, 1047, 12, 413, 1040),
    ("256x256", True): (3, 1448, 14, 335, 1426),
}


def _rand(seed, *shapes, dtype=torch.bfloat16):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [(torch.randn(shape, generator=gen, device="cuda") * (shape[0] ** -0.5 if len(shape) == 2 else 1.0)).to(dtype) for shape in shapes]


def _close(got, want, kind):
    return (got.double() - want).abs().max() <= TOL[kind]["t"] * want.abs().max()


def test_sizes_take_the_tiles_they_are_about():
    """(needs no GPU)"""
    for op, name in enumerate(LINEAR):
        for tile, size in LINEAR[name].items():
            assert linear_plan(op, *size) == (tile.split(",")[0], 1), (name, tile)
    for (tile, chunks), size in WEIGHT.items():
        got = linear_plan(2, *size)
        assert (got[0], got[1] > 1) == (tile, chunks), (tile, chunks)
    for op, name in enumerate(PROJECT):
        for tile, (B, l_x, H, l_s, rv) in PROJECT[name].items():
            assert project_plan(op, B, l_x, H, 64, l_s, rv) == tile, (name, tile)
    for (tile, chunks), (B, l_x, H, l_s, rv) in PARTIALS.items():
        got = project_plan(2, B, l_x, H, 64, l_s, rv)
        assert (got[2], got[3] > 1) == (tile, chunks), (tile, chunks)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", LINEAR["fwd"])
def test_linear_forward(tile):
    rows, K, N = LINEAR["fwd"][tile]
    a, w = _rand(rows + K, (rows, K), (K, N))
    c = lss.lss_linear_fwd(a, w)
    assert _close(c, a.double() @ w.double(), "bf16")
    u, g = lss.lss_linear_gelu_fwd(a, w)
    assert torch.equal(u, c) and torch.equal(g, lss.lss_gelu_fwd(c))


@pytest.mark.gpu
@pytest.mark.parametrize("tile", LINEAR["bwd_input"])
def test_linear_input_gradient(tile):
    rows, K, N = LINEAR["bwd_input"][tile]
    dc, w, u = _rand(rows + N, (rows, N), (K, N), (rows, K))
    da = lss.lss_linear_bwd_input(dc, w)
    assert _close(da, dc.double() @ w.double().T, "bf16")
    assert torch.equal(lss.lss_linear_bwd_input_gelu(dc, w, u), lss.lss_gelu_bwd(u, da))


@pytest.mark.gpu
@pytest.mark.parametrize("tile,chunks", WEIGHT)
def test_linear_weight_gradient(tile, chunks):
    rows, K, N = WEIGHT[tile, chunks]
    a, dc = _rand(rows + K + N, (rows, K), (rows, N))
    dw = lss.lss_linear_bwd_weight(a, dc)
    assert _close(dw, a.double().T @ dc.double(), "f32")
    assert torch.equal(dw, lss.lss_linear_bwd_weight(a, dc))


@pytest.mark.gpu
@pytest.mark.parametrize("tile", PROJECT["qkv"])
def test_projections(tile):
    B, l_x, H, l_s, rv = PROJECT["qkv"][tile]
    E, s0 = 64 * H, rv - l_s
    x, w_q, w_kv = _rand(l_x, (B, l_x, E), (E, E), (E, 2 * E))
    q, k, v = lss.lss_project_qkv(x, w_q, w_kv, s0, l_s, H)
    for b in range(B):
        kv = x[b].double() @ w_kv.double()
        assert _close(q[b].view(l_s, E), x[b, s0:rv].double() @ w_q.double(), "bf16")
        assert _close(k[b].view(l_x, E), kv[:, :E], "bf16") and _close(v[b].view(l_x, E), kv[:, E:], "bf16")


def _partials(seed, B, l_x, H, rv):
    dk, dv = _rand(seed, (B, l_x, H, 64), (B, l_x, H, 64), dtype=torch.float32)
    for t in (dk, dv):
        t[:, rv:] = float("nan")        # never read
    rounded = torch.cat([t[:, :rv].reshape(B, rv, -1).to(torch.bfloat16).double() for t in (dk, dv)], 2)
    return dk, dv, rounded


@pytest.mark.gpu
@pytest.mark.parametrize("tile", PROJECT["bwd"])
def test_projections_input_gradient(tile):
    B, l_x, H, l_s, rv = PROJECT["bwd"][tile]
    E = 64 * H
    w_q, w_kv, dq = _rand(l_x + 1, (E, E), (E, 2 * E), (B, l_s, H, 64))
    dk, dv, rounded = _partials(l_x, B, l_x, H, rv)
    dx_q, dx = lss.lss_project_bwd(dq, dk, dv, w_q, w_kv, rv)
    assert not dx[:, rv:].any()
    for b in range(B):
        assert _close(dx_q[b], dq[b].reshape(l_s, E).double() @ w_q.double().T, "f32")
        assert _close(dx[b, :rv], rounded[b] @ w_kv.double().T, "f32")


@pytest.mark.gpu
@pytest.mark.parametrize("tile,chunks", PARTIALS)
def test_projections_weight_gradient_of_float_partials(tile, chunks):
    B, l_x, H, l_s, rv = PARTIALS[tile, chunks]
    E = 64 * H
    x, dq = _rand(l_x + 2, (B, l_x, E), (B, l_s, H, 64))
    dk, dv, rounded = _partials(l_x + 3, B, l_x, H, rv)
    dw_q, dw_kv = lss.lss_project_bwd_weight(x, dq, dk, dv, rv - l_s, rv)
    assert _close(dw_kv, sum(x[b, :rv].double().T @ rounded[b] for b in range(B)), "f32")
    assert _close(dw_q, sum(x[b, rv - l_s:rv].double().T @ dq[b].reshape(l_s, E).double() for b in range(B)), "f32")
    assert torch.equal(dw_kv, lss.lss_project_bwd_weight(x, dq, dk, dv, rv - l_s, rv)[1])


# The 256 x 256 tile's loop takes its last two contraction tiles by themselves and goes round three slots of one operand and two of the other: 9 to 13 contraction tiles of
# bf16 and 7 to 9 of floats (chunks of them, the last one shorter), last tiles of one, some and all rows; and the maps' shortest (four tiles; eight of the floats).
# FEW_TILES below has the others.
SHORT = {"qkv": (1, 60001, 4, 100, 59998), "bwd": (1, 60001, 4, 100, 59998)}
LENGTHS = (513, 575, 640, 641, 704, 768, 769, 832)
FLOAT_LENGTHS = (1409, 1472, 1473, 1536, 1600, 1664, 1728)


def test_lengths_take_the_256x256_tile():
    """(needs no GPU)"""
    for op, name in enumerate(SHORT):
        B, l_x, H, l_s, rv = SHORT[name]
        assert project_plan(op, B, l_x, H, 64, l_s, rv) == "256x256", name
    for rows in LENGTHS:
        assert linear_plan(2, rows, 1664, 5248) == ("256x256", 1), rows
    for rv in FLOAT_LENGTHS:
        assert project_plan(2, 3, rv + 10, 14, 64, 335, rv)[2] == "256x256", rv


@pytest.mark.gpu
@pytest.mark.parametrize("rows", LENGTHS)
def test_weight_gradient_of_every_length_of_the_loop(rows):
    a, dc = _rand(rows, (rows, 1664), (rows, 5248))
    assert _close(lss.lss_linear_bwd_weight(a, dc), a.double().T @ dc.double(), "f32")


@pytest.mark.gpu
@pytest.mark.parametrize("rv", FLOAT_LENGTHS)
def test_float_weight_gradient_of_every_length_of_the_loop(rv):
    x, dq = _rand(rv, (3, rv + 10, 896), (3, 335, 14, 64))
    dk, dv, rounded = _partials(rv, 3, rv + 10, 14, rv)
    dw_kv = lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 335, rv)[1]
    assert _close(dw_kv, sum(x[b, :rv].double().T @ rounded[b] for b in range(3)), "f32")


@pytest.mark.gpu
def test_projections_of_the_shortest_contractions_of_the_loop():
    B, l_x, H, l_s, rv = SHORT["qkv"]
    E, s0 = 64 * H, rv - l_s
    x, w_q, w_kv, dq = _rand(l_x, (B, l_x, E), (E, E), (E, 2 * E), (B, l_s, H, 64))
    _, k, v = lss.lss_project_qkv(x, w_q, w_kv, s0, l_s, H)
    kv = x[0].double() @ w_kv.double()
    assert _close(k.view(l_x, E), kv[:, :E], "bf16") and _close(v.view(l_x, E), kv[:, E:], "bf16")
    dk, dv, rounded = _partials(l_x, B, l_x, H, rv)
    dx_q, dx = lss.lss_project_bwd(dq, dk, dv, w_q, w_kv, rv)
    assert _close(dx_q[0], dq[0].reshape(l_s, E).double() @ w_q.double().T, "f32")
    assert _close(dx[0, :rv], rounded[0] @ w_kv.double().T, "f32") and not dx[:, rv:].any()


LONG = {"64x64 in groups": (1, 1709, 6, 1700), "32x32": (1, 1130, 2, 1127)}      # B, l_x, H, rows_valid: float chunks of more than 1536 and 1024 rows


LONG_MAPS = {"64x64 in groups": (1, 1110, 16, 284, 344), "32x32": (1, 300, 16, 60, 120)}       # B, l_x, H, l_s, rows_valid: float contractions of 2048


def test_long_float_contractions_take_their_tiles():
    """(needs no GPU)"""
    for tile, (B, l_x, H, l_s, rv) in LONG_MAPS.items():
        assert project_plan(1, B, l_x, H, 64, l_s, rv) == tile, tile
    for tile, (B, l_x, H, rv) in LONG.items():
        assert project_plan(2, B, l_x, H, 64, 90, rv)[2:4] == (tile, 1), tile


@pytest.mark.gpu
@pytest.mark.parametrize("tile", LONG)
def test_weight_gradient_of_long_float_chunks(tile):
    B, l_x, H, rv = LONG[tile]
    x, dq = _rand(rv, (B, l_x, 64 * H), (B, 90, H, 64))
    dk, dv, rounded = _partials(rv, B, l_x, H, rv)
    dw_kv = lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 90, rv)[1]
    assert _close(dw_kv, sum(x[b, :rv].double().T @ rounded[b] for b in range(B)), "f32")
    assert torch.equal(dw_kv, lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 90, rv)[1])


@pytest.mark.gpu
@pytest.mark.parametrize("tile", LONG_MAPS)
def test_input_gradient_of_long_float_contractions(tile):
    B, l_x, H, l_s, rv = LONG_MAPS[tile]
    E = 64 * H
    w_q, w_kv, dq = _rand(l_x + 5, (E, E), (E, 2 * E), (B, l_s, H, 64))
    dk, dv, rounded = _partials(l_x + 6, B, l_x, H, rv)
    dx_q, dx = lss.lss_project_bwd(dq, dk, dv, w_q, w_kv, rv)
    assert _close(dx_q[0], dq[0].reshape(l_s, E).double() @ w_q.double().T, "f32")
    assert _close(dx[0, :rv], rounded[0] @ w_kv.double().T, "f32") and not dx[:, rv:].any()


# Maps of float partials in the small tiles, whose groups and slots are not those of bf16 operands: (tile, groups, slots, H): B, l_x, l_s, rows_valid.  32 x 32 ones on
# either side of where more groups share a contraction, 832.
FLOAT_MAPS = {("32x64", 4, 2, 16): (1, 209, 40, 200), ("32x64", 4, 2, 32): (1, 79, 33, 70), ("32x32", 4, 4, 6): (1, 49, 33, 40), ("32x32", 8, 2, 8): (1, 49, 33, 40),
              ("64x64 in groups", 4, 2, 32): (1, 209, 40, 200)}


def test_float_maps_take_their_groups_and_slots():
    """(needs no GPU)"""
    for (tile, groups, slots, H), (B, l_x, l_s, rv) in FLOAT_MAPS.items():
        assert (project_plan(1, B, l_x, H, 64, l_s, rv), project_form(1, B, l_x, H, 64, l_s, rv)) == (tile, (groups, slots)), (tile, H)
    bf16 = {"32x32": (4, 4), "32x64": (4, 3), "64x64": (1, 4), "64x64 in groups": (2, 4), "128x128 of eight": (1, 4), "128x128": (1, 2), "256x256": (1, 3)}
    for op, name in enumerate(LINEAR):
        for tile, size in LINEAR[name].items():
            assert linear_form(op, *size) == bf16[tile.split(",")[0]], (name, tile)


@pytest.mark.gpu
@pytest.mark.parametrize("tile,groups,slots,H", FLOAT_MAPS)
def test_input_gradient_of_float_maps(tile, groups, slots, H):
    B, l_x, l_s, rv = FLOAT_MAPS[tile, groups, slots, H]
    E = 64 * H
    w_q, w_kv, dq = _rand(E + 7, (E, E), (E, 2 * E), (B, l_s, H, 64))
    dk, dv, rounded = _partials(E + 8, B, l_x, H, rv)
    dx_q, dx = lss.lss_project_bwd(dq, dk, dv, w_q, w_kv, rv)
    assert _close(dx_q[0], dq[0].reshape(l_s, E).double() @ w_q.double().T, "f32")
    assert _close(dx[0, :rv], rounded[0] @ w_kv.double().T, "f32") and not dx[:, rv:].any()


# dW_kv by chunks of rows on either side of where more groups of wavefronts share a float contraction: (tile, rows_valid): H, groups, slots
FLOAT_CHUNKS = {("64x64 in groups", 832): (6, 2, 4), ("64x64 in groups", 833): (6, 4, 2), ("32x32", 832): (2, 4, 4), ("32x32", 833): (2, 8, 2)}


def test_float_chunks_take_their_groups_and_slots():
    """(needs no GPU)"""
    for (tile, rv), (H, groups, slots) in FLOAT_CHUNKS.items():
        assert project_plan(2, 1, rv + 7, H, 64, 90, rv)[2:4] == (tile, 1) and project_form(2, 1, rv + 7, H, 64, 90, rv) == (groups, slots), (tile, rv)
    # measured shorter with four groups, 15.2 us instead of 15.8
    assert project_plan(2, 1, 1352, 6, 64, 90, 1352)[2:4] == ("64x64 in groups", 1) and project_form(2, 1, 1352, 6, 64, 90, 1352) == (4, 2)


@pytest.mark.gpu
@pytest.mark.parametrize("tile,rv", FLOAT_CHUNKS)
def test_weight_gradient_where_groups_change(tile, rv):
    E = 64 * FLOAT_CHUNKS[tile, rv][0]
    x, dq = _rand(rv + E, (1, rv + 7, E), (1, 90, E // 64, 64))
    dk, dv, rounded = _partials(rv + E, 1, rv + 7, E // 64, rv)
    dw_kv = lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 90, rv)[1]
    assert _close(dw_kv, x[0, :rv].double().T @ rounded[0], "f32")
    assert torch.equal(dw_kv, lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 90, rv)[1])


# Weight gradients in 256 x 256 tiles of few contraction tiles (two never enter the loop's body) and the lengths modulo 6 that LENGTHS leaves out, ragged rows and whole ones, tiles
# that end outside the matrix: rows: contraction tiles.  Floats: rows_valid: B, H, contraction tiles, in one chunk.
FEW_TILES = {100: 2, 128: 2, 190: 3, 250: 4, 300: 5, 896: 14}
FEW_FLOAT_TILES = {66: (3, 24, 2), 128: (3, 24, 2), 129: (3, 24, 3), 213: (2, 24, 4), 276: (2, 24, 5), 384: (2, 24, 6), 591: (2, 24, 10)}


def test_few_contraction_tiles_take_the_256x256_tile():
    """(needs no GPU)"""
    for rows, tiles in FEW_TILES.items():
        assert linear_plan(2, rows, 1920, 8064) == ("256x256", 1) and -(-rows // 64) == tiles, rows
    for rv, (B, H, tiles) in FEW_FLOAT_TILES.items():
        assert project_plan(2, B, rv + 10, H, 64, 60, rv)[2:4] == ("256x256", 1) and -(-rv // 64) == tiles, rv
    assert [project_plan(2, 3, rv + 10, 14, 64, 335, rv)[3] for rv in FLOAT_LENGTHS] == [3] * len(FLOAT_LENGTHS)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", FEW_TILES)
def test_weight_gradient_of_few_contraction_tiles(rows):
    a, dc = _rand(rows + 1, (rows, 1920), (rows, 8064))
    assert _close(lss.lss_linear_bwd_weight(a, dc), a.double().T @ dc.double(), "f32")


@pytest.mark.gpu
@pytest.mark.parametrize("rv", FEW_FLOAT_TILES)
def test_float_weight_gradient_of_few_contraction_tiles(rv):
    B, H, _ = FEW_FLOAT_TILES[rv]
    x, dq = _rand(rv + 1, (B, rv + 10, 64 * H), (B, 60, H, 64))
    dk, dv, rounded = _partials(rv + 1, B, rv + 10, H, rv)
    dw_kv = lss.lss_project_bwd_weight(x, dq, dk, dv, rv - 60, rv)[1]
    assert _close(dw_kv, sum(x[b, :rv].double().T @ rounded[b] for b in range(B)), "f32")


# 32-wide tiles whose groups of wavefronts go round their rings, unevenly: (product, tile): rows, K, N, or B, l_x, H, l_s, rows_valid
ROUNDS = {("fwd", "32x64"): (45, 896, 2176), ("fwd", "32x32"): (45, 1152, 384), ("bwd_input", "32x64"): (58, 2176, 896), ("bwd_input", "32x32"): (45, 384, 1152),
          ("weight", "32x64"): (780, 384, 640), ("weight", "32x32"): (1065, 256, 384), ("qkv", "32x64"): (1, 90, 14, 40, 85), ("qkv", "32x32"): (1, 90, 18, 20, 85),
          ("bwd", "32x64"): (1, 409, 6, 33, 400), ("bwd", "32x32"): (1, 99, 10, 33, 90), ("partials", "32x32"): (1, 1130, 2, 90, 1127)}


def test_rounds_are_longer_than_what_is_on_its_way():
    """(needs no GPU)"""
    for (name, tile), size in ROUNDS.items():
        if len(size) == 3:
            op = ("fwd", "bwd_input", "weight").index(name)
            rows, K, N = size
            got, (groups, slots), length = linear_plan(op, *size)[0], linear_form(op, *size), (K, N, rows)[op]
            assert linear_plan(op, *size)[1] == 1
        else:
            op = ("qkv", "bwd", "partials").index(name)
            B, l_x, H, l_s, rv = size
            plan = project_plan(op, B, l_x, H, 64, l_s, rv)
            got, (groups, slots), length = plan[2] if op == 2 else plan, project_form(op, B, l_x, H, 64, l_s, rv), (64 * H, 128 * H, rv)[op]
        tiles = -(-length // 64)
        assert got == tile and tiles > groups * slots and (tiles % groups or name == "bwd"), (name, tile)       # (project_bwd's come in fours)


@pytest.mark.gpu
@pytest.mark.parametrize("name,tile", ROUNDS)
def test_rounds(name, tile):
    size = ROUNDS[name, tile]
    if len(size) == 3:
        rows, K, N = size
        a, w, dc = _rand(rows + K + 3, (rows, K), (K, N), (rows, N))
        if name == "fwd":
            assert _close(lss.lss_linear_fwd(a, w), a.double() @ w.double(), "bf16")
        elif name == "bwd_input":
            assert _close(lss.lss_linear_bwd_input(dc, w), dc.double() @ w.double().T, "bf16")
        else:
            assert _close(lss.lss_linear_bwd_weight(a, dc), a.double().T @ dc.double(), "f32")
        return
    B, l_x, H, l_s, rv = size
    E, s0 = 64 * H, rv - l_s
    x, w_q, w_kv, dq = _rand(l_x + H, (B, l_x, E), (E, E), (E, 2 * E), (B, l_s, H, 64))
    dk, dv, rounded = _partials(l_x + H, B, l_x, H, rv)
    if name == "qkv":
        q, k, v = lss.lss_project_qkv(x, w_q, w_kv, s0, l_s, H)
        kv = x[0].double() @ w_kv.double()
        assert _close(q.view(l_s, E), x[0, s0:rv].double() @ w_q.double(), "bf16")
        assert _close(k.view(l_x, E), kv[:, :E], "bf16") and _close(v.view(l_x, E), kv[:, E:], "bf16")
    elif name == "bwd":
        dx_q, dx = lss.lss_project_bwd(dq, dk, dv, w_q, w_kv, rv)
        assert _close(dx_q[0], dq[0].reshape(l_s, E).double() @ w_q.double().T, "f32")
        assert _close(dx[0, :rv], rounded[0] @ w_kv.double().T, "f32") and not dx[:, rv:].any()
    else:
        assert _close(lss.lss_project_bwd_weight(x, dq, dk, dv, s0, rv)[1], x[0, :rv].double().T @ rounded[0], "f32")

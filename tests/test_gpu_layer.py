"""GPU parity of the segment-local layer operations (Section 3, Principles 1 and 2: positional
embedding row slice, layer normalisation, GeLU, the feed-forward unit) against the fp64 oracle,
through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_02382_amd import lss, synth
from _util import TOL, Staged, rel_err, to_np

pytestmark = pytest.mark.gpu


def staged(seed, shape, kind="bf16", std=1.0, shift=0.0):
    a = synth.normal_f32(seed, int(np.prod(shape))).reshape(shape) * np.float32(std) + np.float32(shift)
    return Staged(a.astype(np.float32), kind)


def assert_rounded(got, ref, tag, slack=1e-4):
    """One rounding to bf16 (2^-9 relative) of a value computed in fp32."""
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, tag
    if ref.size == 0:
        return
    assert np.all(np.isfinite(got)), tag
    bound = 2.0 ** -8 * np.abs(ref) + slack * np.abs(ref).max()
    bad = np.abs(got - ref) > bound
    assert not bad.any(), f"{tag}: {bad.sum()} elements off, worst {np.abs(got - ref).max()}"


PE_SHAPES = [  # B, l_s, l_x, E, s0
    (1, 256, 1024, 256, 256),
    (3, 301, 1000, 512, 437),       # ragged rows, unaligned offset
    (2, 1, 130, 128, 129),          # one row: the last of the table
    (4, 700, 700, 1024, 0),         # the segment is the whole sequence
    (2, 77, 200, 8, 100),           # one 16-byte chunk per row
]


@pytest.mark.parametrize("B,l_s,l_x,E,s0", PE_SHAPES)
def test_embed_pe_matches_oracle(B, l_s, l_x, E, s0):
    TOK, PE = staged(7100 + l_s, (B, l_s, E)), staged(7101 + l_s, (l_x, E))
    x = lss.lss_embed_pe_fwd(TOK.dev, PE.dev, s0)
    assert_rounded(to_np(x), oracle.embed_pe(TOK.f64, PE.f64, s0), f"x {B, l_s, l_x, E, s0}", slack=0.0)
    DX = staged(7102 + l_s, (B, l_s, E))
    dpe = lss.lss_embed_pe_bwd(DX.dev)
    ref = oracle.embed_pe_bwd(DX.f64)
    assert dpe.dtype == torch.float32
    assert rel_err(to_np(dpe), ref) <= 1e-6


def test_embed_pe_segments_tile_the_table():
    # Principle 2: the segments' slices together are the whole table, each row used once
    B, l_x, E, N = 2, 600, 128, 4
    TOK, PE = staged(7110, (B, l_x, E)), staged(7111, (l_x, E))
    whole = lss.lss_embed_pe_fwd(TOK.dev, PE.dev, 0)
    l_s = l_x // N
    for i in range(N):
        part = lss.lss_embed_pe_fwd(TOK.dev[:, i * l_s:(i + 1) * l_s].contiguous(), PE.dev, i * l_s)
        assert torch.equal(part, whole[:, i * l_s:(i + 1) * l_s])


@pytest.mark.parametrize("B,l_s,E,s0,p", [(2, 300, 512, 437, 0.1), (1, 1, 8, 50111, 0.5), (3, 77, 1024, 0, 0.25),
                                          (2, 129, 136, 1000, 0.0)])
def test_residual_dropout_add_matches_oracle(B, l_s, E, s0, p):
    X, DL = staged(7150 + l_s, (B, l_s, E)), staged(7151 + l_s, (B, l_s, E))
    seed = 0xABCD_0000_1234 + l_s
    out = lss.lss_residual_dropout_add(X.dev, DL.dev, s0, p, seed)
    ref = oracle.residual_dropout_add(X.f64, DL.f64, s0, p, seed)
    assert_rounded(to_np(out), ref, f"residual {B, l_s, E, s0, p}", slack=1e-6)
    # the keep decisions are exactly the oracle's: where it dropped, out is x itself
    dropped = oracle.residual_dropout_add(None, np.ones((B, l_s, E)), s0, p, seed) == 0
    assert np.array_equal(to_np(out)[dropped], X.f64[dropped])
    # the branch alone (x absent), which is also the backward of the branch; in place
    alone = lss.lss_residual_dropout_add(None, DL.dev, s0, p, seed)
    assert_rounded(to_np(alone), oracle.residual_dropout_add(None, DL.f64, s0, p, seed), "branch alone", slack=1e-6)
    assert np.array_equal(to_np(alone) == 0, dropped | (DL.f64 == 0))
    buf = X.dev.clone()
    lss.lss_residual_dropout_add(buf, DL.dev, s0, p, seed, out=buf)
    assert torch.equal(buf, out)


LN_SHAPES = [  # rows, E
    (256, 256), (1000, 512), (1, 1024), (333, 2048), (67, 4096), (129, 8), (35, 520), (4100, 128),
]


@pytest.mark.parametrize("rows,E", LN_SHAPES)
def test_layernorm_matches_oracle(rows, E):
    X = staged(7200 + E, (rows, E), std=1.5, shift=0.75)        # a mean the variance must not see
    G, Bt = staged(7201 + E, (E,), "f32", std=0.5, shift=1.0), staged(7202 + E, (E,), "f32", std=0.3)
    y, mean, rstd = lss.lss_layernorm_fwd(X.dev, G.dev, Bt.dev)
    ry, rmean, rrstd = oracle.layernorm_fwd(X.f64, G.f64, Bt.f64)
    assert rel_err(to_np(mean), rmean, floor=1.0) <= 1e-5
    assert rel_err(to_np(rstd), rrstd) <= 1e-5
    assert_rounded(to_np(y), ry, f"y {rows, E}")
    DY = staged(7203 + E, (rows, E))
    dx, dg, db = lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, DY.dev)
    rdx, rdg, rdb = oracle.layernorm_bwd(X.f64, G.f64, DY.f64)
    assert rel_err(to_np(dx), rdx) <= TOL["bf16"]["t"]
    assert_rounded(to_np(dx), rdx, f"dx {rows, E}", slack=2e-4)
    assert rel_err(to_np(dg), rdg) <= 1e-4 and rel_err(to_np(db), rdb) <= 1e-4


def test_layernorm_is_reproducible_and_checks_scratch():
    rows, E = 777, 512
    X, DY = staged(7210, (rows, E)), staged(7211, (rows, E))
    G, Bt = staged(7212, (E,), "f32", shift=1.0), staged(7213, (E,), "f32")
    y, mean, rstd = lss.lss_layernorm_fwd(X.dev, G.dev, Bt.dev)
    a = lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, DY.dev)
    need = lss.lss_layernorm_bwd_scratch_bytes(rows, E)
    assert need == ((rows + 31) // 32) * 2 * E * 4
    scratch = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")      # stale contents must not matter
    b = lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, DY.dev, scratch=scratch)
    for u, v in zip(a, b):
        assert torch.equal(u, v)
    with pytest.raises(lss.LssError) as e:
        lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, DY.dev, scratch=scratch[: need - 16])
    assert e.value.code == -6
    # no rows: parameter gradients are zero
    empty = torch.empty((0, E), dtype=torch.bfloat16, device="cuda")
    none = torch.empty((0,), dtype=torch.float32, device="cuda")
    dx, dg, db = lss.lss_layernorm_bwd(empty, G.dev, none, none, empty,
                                       dgamma=torch.full((E,), 3.0, device="cuda"), dbeta=torch.full((E,), 3.0, device="cuda"))
    assert dx.numel() == 0 and not dg.any() and not db.any()


@pytest.mark.parametrize("rows,E", [(1, 8), (33, 136), (64, 1928), (95, 4096)])
def test_layernorm_backward_in_place(rows, E):
    X, DY = staged(7220, (rows, E)), staged(7221, (rows, E))
    G, Bt = staged(7222, (E,), "f32", shift=1.0), staged(7223, (E,), "f32")
    _, mean, rstd = lss.lss_layernorm_fwd(X.dev, G.dev, Bt.dev)
    want = lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, DY.dev)
    x, dy = X.dev.clone(), DY.dev.clone()
    for got in (lss.lss_layernorm_bwd(X.dev, G.dev, mean, rstd, dy, dx=dy), lss.lss_layernorm_bwd(x, G.dev, mean, rstd, DY.dev, dx=x)):
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    rdx, rdg, rdb = oracle.layernorm_bwd(X.f64, G.f64, DY.f64)
    assert rel_err(to_np(want[0]), rdx) <= TOL["bf16"]["t"] and rel_err(to_np(want[1]), rdg) <= 1e-4 and rel_err(to_np(want[2]), rdb) <= 1e-4


@pytest.mark.parametrize("n", [8, 1000 * 8, 257 * 1024])
def test_gelu_matches_oracle(n):
    U, DG = staged(7300 + n % 97, (n,), std=2.0), staged(7301 + n % 97, (n,))
    g = lss.lss_gelu_fwd(U.dev)
    assert_rounded(to_np(g), oracle.gelu(U.f64), f"gelu {n}", slack=1e-6)
    du = lss.lss_gelu_bwd(U.dev, DG.dev)
    assert_rounded(to_np(du), DG.f64 * oracle.gelu_grad(U.f64), f"gelu' {n}", slack=1e-6)


def test_gelu_tails():
    # far tails: GeLU(u) -> u and -> -0, its derivative -> 1 and -> 0; no NaN from exp/erf
    u = np.array([-40.0, -12.0, -6.0, -1e-3, 0.0, 1e-3, 6.0, 12.0], dtype=np.float32)
    U, DG = Staged(u, "bf16"), Staged(np.ones_like(u), "bf16")
    assert_rounded(to_np(lss.lss_gelu_fwd(U.dev)), oracle.gelu(U.f64), "tails", slack=1e-7)
    assert_rounded(to_np(lss.lss_gelu_bwd(U.dev, DG.dev)), oracle.gelu_grad(U.f64), "tails'", slack=1e-7)


FFN_SHAPES = [  # rows, E, F
    (256, 256, 1024),
    (1000, 128, 512),       # ragged rows; one column tile of the input width
    (1, 384, 1536),         # a single row; widths that are not multiples of 256
    (2300, 512, 2048),      # nine row tiles; several column tiles
    (130, 1024, 128),       # narrower hidden width than input
]


@pytest.mark.parametrize("rows,E,F", FFN_SHAPES)
def test_ffn_matches_oracle(rows, E, F):
    Hh = staged(7400 + rows, (rows, E))
    W1, W2 = staged(7401 + rows, (E, F), std=E ** -0.5), staged(7402 + rows, (F, E), std=F ** -0.5)
    DY = staged(7403 + rows, (rows, E))
    ry, ru = oracle.ffn_fwd(Hh.f64, W1.f64, W2.f64)
    u = lss.lss_linear_fwd(Hh.dev, W1.dev)
    assert_rounded(to_np(u), ru, f"u {rows, E, F}")
    g = lss.lss_gelu_fwd(u)
    y = lss.lss_linear_fwd(g, W2.dev)
    assert rel_err(to_np(y), ry) <= TOL["bf16"]["t"]
    # backward, from the device's own u (bf16): the oracle gets exactly that u
    ru_dev = to_np(u)
    rdh = oracle.ffn_bwd(DY.f64, ru_dev, W1.f64, W2.f64)
    dg = lss.lss_linear_bwd_input(DY.dev, W2.dev)
    assert_rounded(to_np(dg), DY.f64 @ W2.f64.T, f"dg {rows, E, F}")
    du = lss.lss_gelu_bwd(u, dg)
    dh = lss.lss_linear_bwd_input(du, W1.dev)
    assert rel_err(to_np(dh), rdh) <= TOL["bf16"]["t"]


@pytest.mark.parametrize("rows,E,F", FFN_SHAPES)
def test_fused_gelu_forms_equal_the_separate_calls(rows, E, F):
    Hh = staged(7600 + rows, (rows, E))
    W1, W2 = staged(7601 + rows, (E, F), std=E ** -0.5), staged(7602 + rows, (F, E), std=F ** -0.5)
    DY = staged(7603 + rows, (rows, E))
    u = lss.lss_linear_fwd(Hh.dev, W1.dev)
    g = lss.lss_gelu_fwd(u)
    u2, g2 = lss.lss_linear_gelu_fwd(Hh.dev, W1.dev)
    assert torch.equal(u, u2) and torch.equal(g, g2)
    du = lss.lss_gelu_bwd(u, lss.lss_linear_bwd_input(DY.dev, W2.dev))
    du2 = lss.lss_linear_bwd_input_gelu(DY.dev, W2.dev, u)
    assert torch.equal(du, du2)
    # and the fused chain against the oracle, end to end
    y = lss.lss_linear_fwd(g2, W2.dev)
    dh = lss.lss_linear_bwd_input(du2, W1.dev)
    ry, _ = oracle.ffn_fwd(Hh.f64, W1.f64, W2.f64)
    assert rel_err(to_np(y), ry) <= TOL["bf16"]["t"]
    assert rel_err(to_np(dh), oracle.ffn_bwd(DY.f64, to_np(u), W1.f64, W2.f64)) <= TOL["bf16"]["t"]


WGRAD_SHAPES = [  # rows, K, N
    (1, 128, 128), (63, 128, 256), (64, 256, 128), (65, 384, 128), (1000, 256, 1024), (2300, 512, 2048),
    (5000, 128, 128),       # one output tile: the rows are split into many chunks
    (4097, 1024, 384),
]


@pytest.mark.parametrize("rows,K,N", WGRAD_SHAPES)
def test_linear_weight_gradient_matches_oracle(rows, K, N):
    A, DC = staged(7700 + rows, (rows, K)), staged(7701 + rows, (rows, N))
    need = lss.lss_linear_bwd_weight_scratch_bytes(rows, K, N)
    scratch = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device="cuda")     # NaN patterns: must be overwritten
    dw = lss.lss_linear_bwd_weight(A.dev, DC.dev, scratch=scratch)
    assert dw.dtype == torch.float32 and tuple(dw.shape) == (K, N)
    assert rel_err(to_np(dw), oracle.linear_bwd_weight(A.f64, DC.f64)) <= TOL["f32"]["t"]
    again = lss.lss_linear_bwd_weight(A.dev, DC.dev)
    assert torch.equal(dw, again)                       # fixed-order sum of the chunks: bit-reproducible
    if need:
        with pytest.raises(lss.LssError) as e:
            lss.lss_linear_bwd_weight(A.dev, DC.dev, scratch=scratch[: need - 16])
        assert e.value.code == -6


def test_linear_weight_gradient_sums_over_segments_and_handles_no_rows():
    # Section 4: the segments' contributions add up to the whole sequence's gradient
    B, l_x, K, N, n_seg = 2, 900, 256, 384, 3
    A, DC = staged(7710, (B, l_x, K)), staged(7711, (B, l_x, N))
    whole = oracle.linear_bwd_weight(A.f64, DC.f64)
    l_s = l_x // n_seg
    total = sum(to_np(lss.lss_linear_bwd_weight(A.dev[:, i * l_s:(i + 1) * l_s].contiguous(),
                                                DC.dev[:, i * l_s:(i + 1) * l_s].contiguous())) for i in range(n_seg))
    assert rel_err(total, whole) <= TOL["f32"]["t"]
    none = torch.empty((0, K), dtype=torch.bfloat16, device="cuda")
    dw = lss.lss_linear_bwd_weight(none, torch.empty((0, N), dtype=torch.bfloat16, device="cuda"),
                                   dw=torch.full((K, N), 5.0, device="cuda"))
    assert not dw.any()


def test_ffn_weight_gradients_match_oracle():
    rows, E, F = 700, 256, 1024
    Hh, DY = staged(7720, (rows, E)), staged(7721, (rows, E))
    W1, W2 = staged(7722, (E, F), std=E ** -0.5), staged(7723, (F, E), std=F ** -0.5)
    u, g = lss.lss_linear_gelu_fwd(Hh.dev, W1.dev)
    du = lss.lss_linear_bwd_input_gelu(DY.dev, W2.dev, u)
    dw2 = lss.lss_linear_bwd_weight(g, DY.dev)
    dw1 = lss.lss_linear_bwd_weight(Hh.dev, du)
    ru = to_np(u)       # the device's own pre-activation, as the other operand the oracle's
    rg = oracle.gelu(ru)
    assert rel_err(to_np(dw2), oracle.linear_bwd_weight(rg, DY.f64)) <= TOL["bf16"]["t"]
    rdu = (DY.f64 @ W2.f64.T) * oracle.gelu_grad(ru)
    assert rel_err(to_np(dw1), oracle.linear_bwd_weight(Hh.f64, rdu)) <= TOL["bf16"]["t"]


def test_linear_outputs_preallocated_and_on_a_side_stream():
    rows, E, F = 600, 256, 512
    A, W = staged(7500, (rows, E)), staged(7501, (E, F), std=E ** -0.5)
    ref = lss.lss_linear_fwd(A.dev, W.dev)
    st = torch.cuda.Stream()
    c = torch.full((rows, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        lss.lss_linear_fwd(A.dev, W.dev, c=c, stream=st)
    st.synchronize()
    assert torch.equal(c, ref)


def test_layer_operations_at_the_lx24k_segment_size():
    """One lx24k segment (16384 rows, E_m = 1024, inner width 4096) through the calls bench.py --layer-ops
    times; sampled rows against the oracle (every operation here but the weight gradient acts row by
    row), sampled columns of the weight gradients against the oracle's full sum over rows."""
    B, l_s, l_x, E, F, s0 = 4, 4096, 24576, 1024, 4096, 5 * 4096
    rows = B * l_s
    TOKS, PE = staged(7800, (B, l_s, E)), staged(7801, (l_x, E))
    G, Bt = staged(7802, (E,), "f32", std=0.1, shift=1.0), staged(7803, (E,), "f32", std=0.1)
    W1, W2 = staged(7804, (E, F), std=E ** -0.5), staged(7805, (F, E), std=F ** -0.5)
    DY = staged(7806, (B, l_s, E))
    p, seed = 0.1, 3000
    x = lss.lss_embed_pe_fwd(TOKS.dev, PE.dev, s0)
    h, mean, rstd = lss.lss_layernorm_fwd(x, G.dev, Bt.dev)
    u = lss.lss_linear_fwd(h, W1.dev)
    g = lss.lss_gelu_fwd(u)
    y = lss.lss_linear_fwd(g, W2.dev)
    x2 = lss.lss_residual_dropout_add(x, y, s0, p, seed)
    dyb = lss.lss_residual_dropout_add(None, DY.dev, s0, p, seed)
    dg = lss.lss_linear_bwd_input(dyb, W2.dev)
    du = lss.lss_gelu_bwd(u, dg)
    dh = lss.lss_linear_bwd_input(du, W1.dev)
    dw2 = lss.lss_linear_bwd_weight(g, dyb)
    dw1 = lss.lss_linear_bwd_weight(h, du)
    dx, dgam, dbet = lss.lss_layernorm_bwd(x, G.dev, mean, rstd, dh)
    dx = lss.lss_residual_dropout_add(DY.dev, dx, s0)
    dpe = lss.lss_embed_pe_bwd(dx)
    torch.cuda.synchronize()

    rng = np.random.default_rng(7)
    rs = np.unique(np.concatenate([[0, l_s - 1, 255, 256], rng.integers(0, l_s, 12)]))
    t = TOL["bf16"]["t"]
    for b in (0, B - 1):
        sel = lambda a: to_np(a[b, rs])
        # forward chain on the sampled rows, each stage from the device's own input to it
        rx = oracle.embed_pe(TOKS.f64[b:b + 1, rs], PE.f64[s0 + rs], 0)[0]
        assert_rounded(sel(x), rx, "x", slack=0.0)
        rh, rmean, _ = oracle.layernorm_fwd(sel(x), G.f64, Bt.f64)
        assert_rounded(sel(h), rh, "h")
        assert rel_err(to_np(mean.view(B, l_s)[b, rs]), rmean, floor=1.0) <= 1e-5
        ry, ru = oracle.ffn_fwd(sel(h), W1.f64, W2.f64)
        assert_rounded(sel(u), ru, "u")
        assert rel_err(sel(y), ry) <= t
        for j, r in enumerate(rs):      # the residual's keep decisions are those of global row s0 + r
            # (batch entry b keys the generator: the oracle is evaluated with b entries of padding in front)
            pad = np.zeros((b + 1, 1, E))
            pad[b] = sel(y)[j]
            ref = oracle.residual_dropout_add(None, pad, s0 + int(r), p, seed)[b, 0] + sel(x)[j]
            assert_rounded(sel(x2)[j], ref, "x2", slack=1e-6)
        # backward chain
        assert_rounded(sel(dg), sel(dyb) @ W2.f64.T, "dg")
        assert_rounded(sel(du), sel(dg) * oracle.gelu_grad(sel(u)), "du", slack=1e-6)
        assert_rounded(sel(dh), sel(du) @ W1.f64.T, "dh")
    # weight gradients: eight sampled columns, the full sum over 16384 rows
    cols = rng.integers(0, E, 8)
    ref = oracle.linear_bwd_weight(to_np(g.view(rows, F)), to_np(dyb.view(rows, E))[:, cols])
    assert rel_err(to_np(dw2[:, cols]), ref) <= TOL["f32"]["t"]
    cols = rng.integers(0, F, 8)
    ref = oracle.linear_bwd_weight(to_np(h.view(rows, E)), to_np(du.view(rows, F))[:, cols])
    assert rel_err(to_np(dw1[:, cols]), ref) <= TOL["f32"]["t"]
    # sums over all rows: parameter gradients of the layer normalisation, and the table rows
    rdx, rdg, rdb = oracle.layernorm_bwd(to_np(x), G.f64, to_np(dh))
    assert rel_err(to_np(dgam), rdg) <= 1e-4 and rel_err(to_np(dbet), rdb) <= 1e-4
    assert rel_err(to_np(dpe), oracle.embed_pe_bwd(to_np(dx))) <= 1e-6

"""What is measured of this library: the calls a training program of a sequence-parallel transformer makes.

Four kinds of pass, each through the public binding (`paper_2311_02382_amd.lss`) with the buffers such a program keeps:

  sweep      every segment of a sequence forward and backward, then the sums of the dK and dV partials
  segment    one GPU's share: one segment's forward and backward against the whole K and V
  projected  one GPU's share of an attention layer: Q, K, V projections from the gathered x, attention forward and
             backward, the gradients of x and of the projection weights
  layer      the segment-local rest of a layer: positional rows, layer normalisation, feed-forward unit, residual with
             dropout, forward and backward with every gradient

Sizes of the listed cases are the configurations of `synth.WORKLOADS`.  Inputs are i.i.d. Gaussian activations on the
GPU, as those workloads draw them.
"""
from __future__ import annotations

import math

import torch

from paper_2311_02382_amd import lss, synth


def _sizes(name):
    w = synth.WORKLOADS[name]
    return {"B": w.B, "l_x": w.l_x, "l_s": w.l_s, "H": w.H, "d": w.d, "causal": w.causal, "std": w.qkv_std}


def _attention(kind, name, segment=0, dtype="bf16", p_drop=0.0, skip_tail=False):
    c = {"kind": kind, **_sizes(name), "dtype": dtype, "p_drop": p_drop}
    if kind != "sweep":
        c["seg_offset"] = segment * c["l_s"]
    if kind == "segment":
        c["skip_tail"] = skip_tail
    return c


def _layer(name, segment, fused):
    w = synth.WORKLOADS[name]
    return {"kind": "layer", "B": w.B, "l_x": w.l_x, "l_s": w.l_s, "seg_offset": segment * w.l_s, "E": w.H * w.d,
            "p_hidden": 0.1, "fused": fused}


def listed():
    return [
        # the smallest model run, as in a test or a first try: ten calls of a few microseconds each
        {"name": "sweep tiny", **_attention("sweep", "tiny")},
        # an ordinary training sequence, and the benchmark's
        {"name": "sweep lx8k", **_attention("sweep", "lx8k")},
        {"name": "sweep lx24k", **_attention("sweep", "lx24k")},
        # regularised training: dropout on the attention weights
        {"name": "sweep lx8k dropout", **_attention("sweep", "lx8k", p_drop=0.1)},
        # single precision, as the paper's own runs
        {"name": "sweep lx8k f32", **_attention("sweep", "lx8k", dtype="f32")},
        # heads of width 128, not causal (an encoder): every segment costs the same
        {"name": "segment lx32k_d128", **_attention("segment", "lx32k_d128", 15)},
        # ragged rows (1044) and an offset no tile divides, in the middle of a 50k sequence
        {"name": "segment lx50k", **_attention("segment", "lx50k", 24)},
        # 58 rows per GPU, the shortest segments of the paper's largest runs; the sum is told which rows hold data
        {"name": "segment lx50k_skinny", **_attention("segment", "lx50k_skinny", 431, skip_tail=True)},
        # one GPU's share of an attention layer with its projections, at a small and a large model width
        {"name": "projected lx8k", **_attention("projected", "lx8k", 7)},
        {"name": "projected lx24k", **_attention("projected", "lx24k", 5)},
        # the rest of the layer; with short segments GeLU goes into the maps' own calls to save launches
        {"name": "layer lx8k", **_layer("lx8k", 3, True)},
        {"name": "layer lx24k", **_layer("lx24k", 3, False)},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_BUDGET = {"bf16": 1.4e13, "f32": 1.0e12}      # flops: the lx24k sweep does 1.5e13; fp32 matrix cores are slower


def draw(rng):
    while True:
        kind = rng.choice(["sweep", "segment", "segment", "projected", "layer"])
        B = rng.choice([1, 1, 2, 3, 4])
        l_x = _log_int(rng, 512, 50112)
        l_s = min(l_x, _log_int(rng, 58, 4096))
        seg_offset = rng.randint(0, l_x - l_s)
        if kind == "layer":
            return {"kind": kind, "B": B, "l_x": l_x, "l_s": l_s, "seg_offset": seg_offset, "E": 128 * rng.randint(2, 16),
                    "p_hidden": 0.1, "fused": rng.random() < 0.5}
        d = rng.choice([64, 64, 128])
        c = {"kind": kind, "B": B, "l_x": l_x, "l_s": l_s, "H": rng.randint(2, 16), "d": d, "causal": rng.random() < 0.8,
             "std": rng.choice([1.0, 0.125]), "dtype": "bf16", "p_drop": 0.0}
        if kind == "projected":
            c["H"] = 2 * rng.randint(1, 8)         # E_m a multiple of 128
        elif rng.random() < 0.2:
            c["dtype"] = "f32"
        if rng.random() < 0.2:
            c["p_drop"] = 0.1
        if kind == "sweep":
            if -(-l_x // l_s) > 16:                 # partials of every segment are held until their sum
                continue
        else:
            c["seg_offset"] = seg_offset
        if kind == "segment":
            c["skip_tail"] = rng.random() < 0.3
        if work(c)["flops"] * (2.5 if c["p_drop"] else 1.0) <= _BUDGET[c["dtype"]]:
            return c


def _segments(c):
    """(first row, rows) of every segment the pass runs; a sweep's last segment is what is left."""
    if c["kind"] != "sweep":
        return [(c["seg_offset"], c["l_s"])]
    return [(s0, min(c["l_s"], c["l_x"] - s0)) for s0 in range(0, c["l_x"], c["l_s"])]


def _rows_valid(c, s0, l_s):
    return s0 + l_s if c["causal"] else c["l_x"]


def _normal(gen, shape, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std).to(dtype)


def _empty(shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _prepare_layer(c, gen):
    B, l_s, E, F = c["B"], c["l_s"], c["E"], 4 * c["E"]
    rows = B * l_s
    s = {"tok": _normal(gen, (B, l_s, E)), "pe": _normal(gen, (c["l_x"], E)), "w1": _normal(gen, (E, F), E ** -0.5),
         "w2": _normal(gen, (F, E), F ** -0.5), "dy": _normal(gen, (B, l_s, E)),
         "gamma": 1.0 + _normal(gen, (E,), 0.1, torch.float32), "beta": _normal(gen, (E,), 0.1, torch.float32)}
    for name in ("x", "h", "y", "x2", "dyb", "dh", "dx"):
        s[name] = _empty((B, l_s, E), torch.bfloat16)
    for name in ("u", "g", "dg", "du"):
        s[name] = _empty((B, l_s, F), torch.bfloat16)
    s.update(mean=_empty((rows,)), rstd=_empty((rows,)), dgamma=_empty((E,)), dbeta=_empty((E,)), dpe=_empty((l_s, E)),
             dw1=_empty((E, F)), dw2=_empty((F, E)))
    s["ln_scratch"] = _empty((max(16, lss.lss_layernorm_bwd_scratch_bytes(rows, E)),), torch.uint8)
    s["w_scratch"] = _empty((max(16, lss.lss_linear_bwd_weight_scratch_bytes(rows, E, F),
                                 lss.lss_linear_bwd_weight_scratch_bytes(rows, F, E)),), torch.uint8)
    return s


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if c["kind"] == "layer":
        return {"case": c, "seed": seed, **_prepare_layer(c, gen)}
    B, l_x, H, d = c["B"], c["l_x"], c["H"], c["d"]
    E, dt = H * d, torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    segs = _segments(c)
    s = {"case": c, "segs": segs, "drop": {"p_drop": c["p_drop"], "seed": seed} if c["p_drop"] else {}}
    if c["kind"] == "projected":
        s["x"] = _normal(gen, (B, l_x, E))
        s["w_q"], s["w_kv"] = _normal(gen, (E, E), c["std"] * E ** -0.5), _normal(gen, (E, 2 * E), c["std"] * E ** -0.5)
        s["q"] = [_empty((B, n, H, d), dt) for _, n in segs]
        s["k"], s["v"] = _empty((B, l_x, H, d), dt), _empty((B, l_x, H, d), dt)
        l_s = c["l_s"]
        s["dx_q"], s["dx_partial"] = _empty((B, l_s, E)), _empty((B, l_x, E))
        s["dw_q"], s["dw_kv"] = _empty((E, E)), _empty((E, 2 * E))
        s["w_scratch"] = _empty((max(16, lss.lss_project_bwd_weight_scratch_bytes(l_s, l_x, B, H, d)),), torch.uint8)
    else:
        s["q"] = [_normal(gen, (B, n, H, d), c["std"], dt) for _, n in segs]
        s["k"], s["v"] = _normal(gen, (B, l_x, H, d), c["std"], dt), _normal(gen, (B, l_x, H, d), c["std"], dt)
    s["d_out"] = [_normal(gen, (B, n, H, d), 1.0, dt) for _, n in segs]
    s["out"], s["dq"] = [torch.empty_like(t) for t in s["d_out"]], [torch.empty_like(t) for t in s["d_out"]]
    s["lse"] = [_empty((B, H, n)) for _, n in segs]
    # with skip_tail the rows no query sees stay as the program last left them: here zeros
    new = torch.zeros if c.get("skip_tail") else torch.empty
    s["dk_part"], s["dv_part"] = ([new((B, l_x, H, d), dtype=torch.float32, device="cuda") for _ in segs] for _ in range(2))
    if c["kind"] == "sweep":
        s["dk"], s["dv"] = _empty((B, l_x, H, d)), _empty((B, l_x, H, d))
        s["rows_valid"] = [_rows_valid(c, s0, n) for s0, n in segs]
    return s


def _run_layer(s):
    c = s["case"]
    s0, p, seed = c["seg_offset"], c["p_hidden"], s["seed"]
    lss.lss_embed_pe_fwd(s["tok"], s["pe"], s0, x=s["x"])
    lss.lss_layernorm_fwd(s["x"], s["gamma"], s["beta"], y=s["h"], mean=s["mean"], rstd=s["rstd"])
    if c["fused"]:
        lss.lss_linear_gelu_fwd(s["h"], s["w1"], u=s["u"], g=s["g"])
    else:
        lss.lss_linear_fwd(s["h"], s["w1"], c=s["u"])
        lss.lss_gelu_fwd(s["u"], g=s["g"])
    lss.lss_linear_fwd(s["g"], s["w2"], c=s["y"])
    lss.lss_residual_dropout_add(s["x"], s["y"], s0, p, seed, out=s["x2"])
    # backward: through the branch's dropout, the feed-forward unit and its weights, the normalisation, the skip path
    lss.lss_residual_dropout_add(None, s["dy"], s0, p, seed, out=s["dyb"])
    if c["fused"]:
        lss.lss_linear_bwd_input_gelu(s["dyb"], s["w2"], s["u"], du=s["du"])
    else:
        lss.lss_linear_bwd_input(s["dyb"], s["w2"], da=s["dg"])
        lss.lss_gelu_bwd(s["u"], s["dg"], du=s["du"])
    lss.lss_linear_bwd_input(s["du"], s["w1"], da=s["dh"])
    lss.lss_linear_bwd_weight(s["g"], s["dyb"], dw=s["dw2"], scratch=s["w_scratch"])
    lss.lss_linear_bwd_weight(s["h"], s["du"], dw=s["dw1"], scratch=s["w_scratch"])
    lss.lss_layernorm_bwd(s["x"], s["gamma"], s["mean"], s["rstd"], s["dh"], dx=s["dx"], dgamma=s["dgamma"], dbeta=s["dbeta"],
                          scratch=s["ln_scratch"])
    lss.lss_residual_dropout_add(s["dy"], s["dx"], s0, 0.0, 0, out=s["dx"])
    lss.lss_embed_pe_bwd(s["dx"], dpe_rows=s["dpe"])
    return {k: s[k] for k in ("x2", "u", "g", "dx", "dw1", "dw2", "dgamma", "dbeta", "dpe")}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "layer":
        return _run_layer(s)
    k, v, causal, drop = s["k"], s["v"], c["causal"], s["drop"]
    for i, (s0, n) in enumerate(s["segs"]):
        if c["kind"] == "projected":
            lss.lss_project_qkv(s["x"], s["w_q"], s["w_kv"], s0, n, c["H"], q_seg=s["q"][i], k=k, v=v)
        lss.lss_segment_attn_fwd(s["q"][i], k, v, s0, causal, out=s["out"][i], lse=s["lse"][i], **drop)
        lss.lss_segment_attn_bwd(s["q"][i], k, v, s0, s["out"][i], s["lse"][i], s["d_out"][i], causal, dq=s["dq"][i],
                                 dk_partial=s["dk_part"][i], dv_partial=s["dv_part"][i],
                                 skip_masked_tail=c.get("skip_tail", False), **drop)
    r = {name: s[name] for name in ("out", "lse", "dq")}
    if c["kind"] == "sweep":
        lss.lss_reduce_partials(s["dk_part"], s["rows_valid"], out=s["dk"])
        lss.lss_reduce_partials(s["dv_part"], s["rows_valid"], out=s["dv"])
        return {**r, "dk": s["dk"], "dv": s["dv"]}
    r.update(dk=s["dk_part"], dv=s["dv_part"])
    if c["kind"] == "projected":
        rv = _rows_valid(c, *s["segs"][0])
        lss.lss_project_bwd(s["dq"][0], s["dk_part"][0], s["dv_part"][0], s["w_q"], s["w_kv"], rv, dx_q=s["dx_q"],
                            dx_partial=s["dx_partial"])
        lss.lss_project_bwd_weight(s["x"], s["dq"][0], s["dk_part"][0], s["dv_part"][0], s["segs"][0][0], rv, dw_q=s["dw_q"],
                                   dw_kv=s["dw_kv"], scratch=s["w_scratch"])
        r.update({name: s[name] for name in ("q", "k", "v", "dx_q", "dx_partial", "dw_q", "dw_kv")})
    return r


def work(case):
    c = case
    if c["kind"] == "layer":
        rows, E, F = c["B"] * c["l_s"], c["E"], 4 * c["E"]
        # in: tok, dy, table rows, both weights, gamma, beta; out: x2, u, g, dx, and the gradients in fp32
        return {"bytes": 2 * (2 * rows * E + c["l_s"] * E + 2 * E * F) + 8 * E + 2 * (2 * rows * E + 2 * rows * F)
                + 4 * (2 * E * F + 2 * E + c["l_s"] * E), "flops": 12 * rows * E * F}
    B, l_x, H, d = c["B"], c["l_x"], c["H"], c["d"]
    E, eb = H * d, 4 if c["dtype"] == "f32" else 2
    pairs = rows = valid = 0
    for s0, n in _segments(c):
        pairs += (n * s0 + n * (n + 1) // 2 if c["causal"] else n * l_x) * B * H
        rows += B * n
        valid = max(valid, B * _rows_valid(c, s0, n))
    flops = 12 * d * pairs
    read = valid                    # key rows some query sees
    written = valid if c.get("skip_tail") else B * l_x
    # q, dO in, out, dq out; k, v in; lse out; the gradients of k and v in fp32
    nbytes = eb * E * (4 * rows + 2 * read) + 4 * H * rows + 8 * E * written
    if c["kind"] == "projected":
        flops += 2 * E * (2 * E * (B * l_x + 2 * valid) + 3 * E * rows)
        # x and the weights in; q, k, v (written here, not read), the gradients of x and of the weights out
        nbytes += eb * E * (B * l_x + 3 * E) + eb * E * 2 * (B * l_x - read) + 4 * E * (rows + B * l_x + 3 * E)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 storage with fp32 accumulation, weights and score gradients rounded to bf16 before their products
    return {"rel": 1e-5} if case.get("dtype") == "f32" else {"rel": 1e-2}

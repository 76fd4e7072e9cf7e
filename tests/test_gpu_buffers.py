"""What a caller may do with the buffers it passes, beyond giving each call its own."""
import pytest
import torch

from paper_2311_02382_amd import lss, timing
from _util import TOL, rel_err, stage_all, to_np

pytestmark = pytest.mark.gpu


def _problem(kind, B, l_x, H, d, s0, l_s, causal, **drop):
    Q, K, V, DO = stage_all(B, l_x, H, d, 9100 + l_s, kind)
    q, do = Q.dev[:, s0:s0 + l_s].contiguous(), DO.dev[:, s0:s0 + l_s].contiguous()
    out, lse = lss.lss_segment_attn_fwd(q, K.dev, V.dev, s0, causal, **drop)
    return q, K.dev, V.dev, do, out, lse


def _launches(kernel, call):
    kid = {n: i for i, n in timing.kernel_names().items()}[kernel]
    timing.reset()
    timing.enable(True)
    try:
        call()
        return timing.read(kid)[1]
    finally:
        timing.enable(False)


OVERWRITES = [  # kind, B, l_x, H, d, s0, l_s, causal, p_drop: row sums within the main launch (each kind of workgroup that does so), ahead of it
    ("bf16", 1, 512, 4, 64, 256, 256, True, 0.0), ("bf16", 1, 640, 3, 128, 333, 200, False, 0.0), ("bf16", 1, 512, 4, 64, 200, 256, True, 0.1),
    ("bf16", 1, 400, 2, 64, 100, 58, True, 0.0), ("bf16", 1, 700, 2, 128, 300, 33, True, 0.0),
    ("bf16", 1, 1403, 20, 64, 1203, 58, True, 0.0), ("bf16", 2, 2001, 32, 64, 1830, 128, True, 0.0),
    ("bf16", 1, 1100, 2, 64, 33, 1029, True, 0.0), ("f32", 1, 600, 2, 64, 100, 300, True, 0.0),
]


@pytest.mark.parametrize("where", ["dq", "dq_shifted", "dk", "dv"])
@pytest.mark.parametrize("kind,B,l_x,H,d,s0,l_s,causal,p_drop", OVERWRITES)
def test_gradients_over_the_output(kind, B, l_x, H, d, s0, l_s, causal, p_drop, where):
    # `out` is dead after the backward: its memory may take a gradient, whole or in part.  Each value of `out` must then
    # have been read before the launch that writes gradients, whichever workgroups would read it otherwise.
    drop = dict(p_drop=p_drop, seed=5) if p_drop else {}
    q, k, v, do, out, lse = _problem(kind, B, l_x, H, d, s0, l_s, causal, **drop)
    want = lss.lss_segment_attn_bwd(q, k, v, s0, out, lse, do, causal, **drop)
    n, shift = out.numel(), 8 * d
    outs = {}
    if where == "dq":
        over = out.clone()
        outs["dq"] = over
    elif where == "dq_shifted":
        buf = torch.zeros(n + shift, dtype=out.dtype, device="cuda")
        over = buf[:n].view_as(out)
        outs["dq"] = buf[shift:].view_as(out)
    else:
        part = torch.zeros(k.shape, dtype=torch.float32, device="cuda")
        over = part.view(-1).view(out.dtype)[:n].view_as(out)
        outs[where + "_partial"] = part
    over.copy_(out)
    got = {}

    def call():
        got["r"] = lss.lss_segment_attn_bwd(q, k, v, s0, over, lse, do, causal, **outs, **drop)
    first = "bwd_prep_bf16_kernel" if kind == "bf16" else "bwd_rowdot_kernel"
    assert _launches(first, call) == 1
    for name, a, b in zip(("dq", "dk", "dv"), got["r"], want):
        assert rel_err(to_np(a), to_np(b)) <= TOL[kind]["t"], name

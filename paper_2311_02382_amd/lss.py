"""Thin binding over liblss_attn.so: same names as the C ABI (include/lss_attn.h).

Argument marshalling only -- every step of the path runs in the HIP kernels.  torch
supplies device memory and the stream; nothing here computes.  The functions below
declare the public signatures; checking the tensors, allocating outputs that were not
passed and calling the library is done in native code (csrc/lss_torch.cpp, built into
_lss_torch): in Python that took 13 us per call, more than the kernels of a short
segment.  If the library has not been built, the first call raises (there is no
fallback path).
"""
from __future__ import annotations

import ctypes
from pathlib import Path

import torch

_PKG = Path(__file__).resolve().parent
LIB_PATH = _PKG / "liblss_attn.so"
_lib = None
_native = None

LSS_OK = 0
STATUS_NAMES = {0: "LSS_OK", -1: "LSS_ERR_NULL", -2: "LSS_ERR_SHAPE", -3: "LSS_ERR_UNSUPPORTED_D",
                -4: "LSS_ERR_ALIGN", -5: "LSS_ERR_RANGE", -6: "LSS_ERR_WORKSPACE", -7: "LSS_ERR_LAUNCH"}

EXPORTS = ["lss_version", "lss_last_error", "lss_workspace_bytes", "lss_set_workspace",
           "lss_segment_attn_fwd", "lss_segment_attn_bwd", "lss_segment_attn_fwd_f32",
           "lss_segment_attn_bwd_f32", "lss_segment_attn_fwd_dropout", "lss_segment_attn_bwd_dropout",
           "lss_segment_attn_fwd_ex", "lss_segment_attn_bwd_ex", "lss_segment_attn_bwd_noalloc", "lss_reduce_partials", "lss_project_qkv", "lss_project_bwd",
           "lss_project_bwd_ex", "lss_project_bwd_weight_scratch_bytes", "lss_project_bwd_weight",
           "lss_embed_pe_fwd", "lss_embed_pe_bwd", "lss_residual_dropout_add", "lss_layernorm_fwd", "lss_layernorm_bwd_scratch_bytes",
           "lss_layernorm_bwd", "lss_linear_fwd", "lss_linear_bwd_input", "lss_linear_bwd_weight_scratch_bytes", "lss_linear_bwd_weight",
           "lss_linear_gelu_fwd",
           "lss_linear_bwd_input_gelu", "lss_gelu_fwd", "lss_gelu_bwd"]

LSS_FLAG_SKIP_MASKED_TAIL = 1


class LssError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"{STATUS_NAMES.get(code, code)}: {msg}")
        self.code = code


def load():
    """Load the built library (once).  Raises if it is missing."""
    global _lib
    if _lib is not None:
        return _lib
    if not LIB_PATH.exists():
        raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2311_02382_amd.build` "
                           "(there is no fallback implementation)")
    lib = ctypes.CDLL(str(LIB_PATH))
    i64, vp, ci, sz = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
    lib.lss_version.restype = ci
    lib.lss_last_error.restype = ctypes.c_char_p
    lib.lss_workspace_bytes.argtypes = [i64, i64, i64, i64, i64, ci]
    lib.lss_workspace_bytes.restype = sz
    lib.lss_set_workspace.argtypes = [vp, sz]
    lib.lss_set_workspace.restype = ci
    fwd = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, vp, vp, vp]
    bwd = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, vp, vp, vp, vp, vp, vp, vp]
    for name, args in (("lss_segment_attn_fwd", fwd), ("lss_segment_attn_fwd_f32", fwd),
                       ("lss_segment_attn_bwd", bwd), ("lss_segment_attn_bwd_f32", bwd),
                       ("lss_segment_attn_bwd_noalloc", bwd)):
        getattr(lib, name).argtypes = args
        getattr(lib, name).restype = ci
    f64, u64 = ctypes.c_double, ctypes.c_uint64
    lib.lss_segment_attn_fwd_dropout.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, f64, u64, ci, vp, vp, vp]
    lib.lss_segment_attn_bwd_dropout.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, f64, u64, ci,
                                                 vp, vp, vp, vp, vp, vp, vp]
    lib.lss_segment_attn_fwd_dropout.restype = ci
    lib.lss_segment_attn_bwd_dropout.restype = ci
    cu = ctypes.c_uint
    lib.lss_segment_attn_fwd_ex.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, f64, u64, ci, cu, vp, sz, vp, vp, vp]
    lib.lss_segment_attn_bwd_ex.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, ci, f64, u64, ci, cu, vp, sz,
                                            vp, vp, vp, vp, vp, vp, vp]
    lib.lss_segment_attn_fwd_ex.restype = ci
    lib.lss_segment_attn_bwd_ex.restype = ci
    lib.lss_reduce_partials.argtypes = [vp, ci, vp, i64, i64, i64, i64, vp, vp]
    lib.lss_reduce_partials.restype = ci
    lib.lss_project_qkv.argtypes = [vp, vp, vp, i64, i64, i64, i64, i64, i64, vp, vp, vp, vp]
    lib.lss_project_qkv.restype = ci
    lib.lss_project_bwd.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, vp, vp, vp]
    lib.lss_project_bwd.restype = ci
    lib.lss_project_bwd_ex.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, cu, vp, vp, vp]
    lib.lss_project_bwd_ex.restype = ci
    lib.lss_project_bwd_weight_scratch_bytes.argtypes = [i64, i64, i64, i64, i64]
    lib.lss_project_bwd_weight_scratch_bytes.restype = sz
    lib.lss_project_bwd_weight.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, vp, vp, vp, sz, vp]
    lib.lss_project_bwd_weight.restype = ci
    lib.lss_embed_pe_fwd.argtypes = [vp, vp, i64, i64, i64, i64, i64, vp, vp]
    lib.lss_embed_pe_bwd.argtypes = [vp, i64, i64, i64, vp, vp]
    lib.lss_residual_dropout_add.argtypes = [vp, vp, i64, i64, i64, i64, f64, u64, vp, vp]
    lib.lss_residual_dropout_add.restype = ci
    lib.lss_layernorm_fwd.argtypes = [vp, vp, vp, f64, i64, i64, vp, vp, vp, vp]
    lib.lss_layernorm_bwd_scratch_bytes.argtypes = [i64, i64]
    lib.lss_layernorm_bwd_scratch_bytes.restype = sz
    lib.lss_layernorm_bwd.argtypes = [vp, vp, vp, vp, vp, i64, i64, vp, vp, vp, vp, sz, vp]
    lib.lss_linear_fwd.argtypes = [vp, vp, i64, i64, i64, vp, vp]
    lib.lss_linear_bwd_input.argtypes = [vp, vp, i64, i64, i64, vp, vp]
    lib.lss_linear_bwd_weight_scratch_bytes.argtypes = [i64, i64, i64]
    lib.lss_linear_bwd_weight_scratch_bytes.restype = sz
    lib.lss_linear_bwd_weight.argtypes = [vp, vp, i64, i64, i64, vp, vp, sz, vp]
    lib.lss_linear_bwd_weight.restype = ci
    lib.lss_linear_gelu_fwd.argtypes = [vp, vp, i64, i64, i64, vp, vp, vp]
    lib.lss_linear_bwd_input_gelu.argtypes = [vp, vp, vp, i64, i64, i64, vp, vp]
    lib.lss_gelu_fwd.argtypes = [vp, i64, vp, vp]
    lib.lss_gelu_bwd.argtypes = [vp, vp, i64, vp, vp]
    for name in ("lss_embed_pe_fwd", "lss_embed_pe_bwd", "lss_residual_dropout_add", "lss_layernorm_fwd", "lss_layernorm_bwd", "lss_linear_fwd",
                 "lss_linear_bwd_input", "lss_linear_gelu_fwd", "lss_linear_bwd_input_gelu", "lss_gelu_fwd", "lss_gelu_bwd"):
        getattr(lib, name).restype = ci
    _lib = lib
    return lib


def _bind():
    """The native half of the binding, loaded once together with the library."""
    global _native
    if _native is None:
        load()
        try:
            from . import _lss_torch
        except ImportError as e:
            raise RuntimeError(f"the native half of the binding cannot be loaded ({e}): build it with `python -m "
                               "paper_2311_02382_amd.build` (there is no fallback implementation)") from e
        if _lss_torch.torch_version != str(torch.__version__):
            raise RuntimeError(f"the native half of the binding was built for torch {_lss_torch.torch_version} and this is torch "
                               f"{torch.__version__}: build it again with `python -m paper_2311_02382_amd.build`")
        _lss_torch.set_error_type(LssError)
        _native = _lss_torch
    return _native


def _check(rc: int):
    if rc != LSS_OK:
        raise LssError(rc, load().lss_last_error().decode())


def lss_version() -> int:
    return int(load().lss_version())


def lss_last_error() -> str:
    return load().lss_last_error().decode()


def lss_workspace_bytes(l_s, l_x, B, H, d, elem_bytes=2) -> int:
    return int(load().lss_workspace_bytes(l_s, l_x, B, H, d, elem_bytes))


def lss_set_workspace(buf) -> None:
    """Hand the library a device buffer (a uint8 torch tensor) as scratch; None clears it."""
    if buf is None:
        _check(load().lss_set_workspace(None, 0))
        return
    _check(load().lss_set_workspace(buf.data_ptr(), buf.numel() * buf.element_size()))


def lss_segment_attn_fwd(q_seg, k, v, seg_offset, causal=True, out=None, lse=None, stream=None,
                         p_drop=None, seed=0, workspace=None):
    """Forward of one segment, bf16 or float32 by the tensors' dtype, through lss_segment_attn_fwd_ex: with dropout when
    p_drop is given, and with scratch of its own when `workspace` (a device tensor of lss_workspace_bytes() bytes
    used by this call alone) is given; otherwise with the binding's buffer of that GPU.

    Returns (out [B,l_s,H,d] in the input dtype, lse [B,H,l_s] float32).
    """
    return (_native or _bind()).attn_fwd(q_seg, k, v, seg_offset, causal, out, lse, stream, p_drop, seed, workspace)


def lss_segment_attn_bwd(q_seg, k, v, seg_offset, out, lse, d_out, causal=True,
                         dq=None, dk_partial=None, dv_partial=None, stream=None, p_drop=None, seed=0,
                         skip_masked_tail=False, workspace=None):
    """Backward of one segment.  Returns (dq, dk_partial, dv_partial); partials are float32 [B,l_x,H,d].

    Through lss_segment_attn_bwd_ex; skip_masked_tail is LSS_FLAG_SKIP_MASKED_TAIL, p_drop, seed and `workspace` as in
    lss_segment_attn_fwd."""
    return (_native or _bind()).attn_bwd(q_seg, k, v, seg_offset, out, lse, d_out, causal, dq, dk_partial, dv_partial, stream, p_drop, seed,
                               skip_masked_tail, workspace)


LSS_NOALLOC_SCRATCH_BYTES = 64 << 20


def lss_segment_attn_bwd_noalloc(q_seg, k, v, seg_offset, out, lse, d_out, causal, dq, dk_partial, dv_partial, stream=None):
    """lss_segment_attn_bwd with the library's built-in scratch buffer (bf16 only): the call itself allocates
    nothing, so every output must be passed in."""
    return (_native or _bind()).attn_bwd_noalloc(q_seg, k, v, seg_offset, out, lse, d_out, causal, dq, dk_partial, dv_partial, stream)


def lss_reduce_partials(parts, rows_valid=None, out=None, stream=None):
    """out = parts[0] + parts[1] + ... in list order; rows >= rows_valid[i] of parts[i] count as 0."""
    return (_native or _bind()).reduce_partials(list(parts), None if rows_valid is None else list(rows_valid), out, stream)


def lss_project_qkv(x, w_q, w_kv, seg_offset, l_s, H, q_seg=None, k=None, v=None, stream=None):
    """Q_i = x_i W_q, K = x W_k, V = x W_v.  x [B,l_x,E] bf16, w_q [E,E], w_kv [E,2E] = [W_k | W_v].

    Returns (q_seg [B,l_s,H,d], k [B,l_x,H,d], v [B,l_x,H,d]) in bf16.
    """
    return (_native or _bind()).project_qkv(x, w_q, w_kv, seg_offset, l_s, H, q_seg, k, v, stream)


def lss_project_bwd(dq, dk_partial, dv_partial, w_q, w_kv, rows_valid=None, dx_q=None, dx_partial=None, stream=None,
                    skip_masked_tail=False):
    """dx_q = dQ_i W_q^T [B,l_s,E] and dx_partial = dK_part W_k^T + dV_part W_v^T [B,l_x,E], both float32.

    Through lss_project_bwd_ex; skip_masked_tail is LSS_FLAG_SKIP_MASKED_TAIL."""
    return (_native or _bind()).project_bwd(dq, dk_partial, dv_partial, w_q, w_kv, rows_valid, dx_q, dx_partial, stream, skip_masked_tail)


def lss_project_bwd_weight_scratch_bytes(l_s, l_x, B, H, d):
    return int(load().lss_project_bwd_weight_scratch_bytes(int(l_s), int(l_x), int(B), int(H), int(d)))


def lss_project_bwd_weight(x, dq, dk_partial, dv_partial, seg_offset, rows_valid=None, dw_q=None, dw_kv=None,
                           scratch=None, stream=None):
    """One segment's share of dW_q [E,E] = sum_b x_i^T dQ_i and dW_kv [E,2E] = sum_b x^T [dK_part | dV_part], float32."""
    return (_native or _bind()).project_bwd_weight(x, dq, dk_partial, dv_partial, seg_offset, rows_valid, dw_q, dw_kv, scratch, stream)


def lss_embed_pe_fwd(tok, pe_table, seg_offset, x=None, stream=None):
    """x[b, r] = tok[b, r] + pe_table[seg_offset + r].  tok [B,l_s,E] bf16, pe_table [l_x,E] bf16."""
    return (_native or _bind()).embed_pe_fwd(tok, pe_table, seg_offset, x, stream)


def lss_embed_pe_bwd(dx, dpe_rows=None, stream=None):
    """dpe_rows[r] = sum_b dx[b, r], float32 [l_s, E]: the gradient of the segment's rows of the table."""
    return (_native or _bind()).embed_pe_bwd(dx, dpe_rows, stream)


def lss_residual_dropout_add(x, delta, seg_offset, p_drop=0.0, seed=0, out=None, stream=None):
    """out = x + dropout(delta) on a segment's rows [B, l_s, E] bf16; x may be None (zeros)."""
    return (_native or _bind()).residual_dropout_add(x, delta, seg_offset, p_drop, seed, out, stream)


def lss_layernorm_fwd(x, gamma, beta, eps=1e-5, y=None, mean=None, rstd=None, stream=None):
    """Row-wise layer normalisation of x [..., E] bf16; returns (y bf16, mean, rstd float32 [rows])."""
    return (_native or _bind()).layernorm_fwd(x, gamma, beta, eps, y, mean, rstd, stream)


def lss_layernorm_bwd_scratch_bytes(rows, E):
    return int(load().lss_layernorm_bwd_scratch_bytes(int(rows), int(E)))


def lss_layernorm_bwd(x, gamma, mean, rstd, dy, dx=None, dgamma=None, dbeta=None, scratch=None, stream=None):
    """Backward of lss_layernorm_fwd: returns (dx bf16, dgamma, dbeta float32 [E]).

    `scratch` is a uint8 device tensor of at least lss_layernorm_bwd_scratch_bytes(rows, E) bytes
    (allocated here if absent).
    """
    return (_native or _bind()).layernorm_bwd(x, gamma, mean, rstd, dy, dx, dgamma, dbeta, scratch, stream)


def lss_linear_fwd(a, w, c=None, stream=None):
    """c = a w.  a [..., K] bf16, w [K, N] bf16 -> c [..., N] bf16."""
    return (_native or _bind()).linear_fwd(a, w, c, stream)


def lss_linear_bwd_input(dc, w, da=None, stream=None):
    """da = dc w^T.  dc [..., N] bf16, w [K, N] bf16 -> da [..., K] bf16."""
    return (_native or _bind()).linear_bwd_input(dc, w, da, stream)


def lss_linear_bwd_weight_scratch_bytes(rows, K, N):
    return int(load().lss_linear_bwd_weight_scratch_bytes(int(rows), int(K), int(N)))


def lss_linear_bwd_weight(a, dc, dw=None, scratch=None, stream=None):
    """dw = a^T dc over every row.  a [..., K], dc [..., N] bf16 -> dw [K, N] float32.

    `scratch` is a uint8 device tensor of at least lss_linear_bwd_weight_scratch_bytes(rows, K, N)
    bytes (allocated here if absent)."""
    return (_native or _bind()).linear_bwd_weight(a, dc, dw, scratch, stream)


def lss_linear_gelu_fwd(a, w, u=None, g=None, stream=None):
    """u = a w and g = GeLU(u) in one kernel; returns (u, g), both [..., N] bf16."""
    return (_native or _bind()).linear_gelu_fwd(a, w, u, g, stream)


def lss_linear_bwd_input_gelu(dc, w, u, du=None, stream=None):
    """du = (dc w^T) * GeLU'(u) in one kernel.  dc [..., N], w [K, N], u [..., K] -> du [..., K], bf16."""
    return (_native or _bind()).linear_bwd_input_gelu(dc, w, u, du, stream)


def lss_gelu_fwd(u, g=None, stream=None):
    """g = GeLU(u) = u Phi(u), elementwise, bf16."""
    return (_native or _bind()).gelu_fwd(u, g, stream)


def lss_gelu_bwd(u, dg, du=None, stream=None):
    """du = dg * GeLU'(u), elementwise, bf16."""
    return (_native or _bind()).gelu_bwd(u, dg, du, stream)

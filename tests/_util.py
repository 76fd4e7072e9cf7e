"""Helpers shared by the GPU parity tests: input staging and the error metrics."""
import collections
import ctypes

import numpy as np
import torch

import oracle
from paper_2311_02382_amd import lss, synth

# Tolerances: max |gpu - ref| / max |ref| per tensor (elementwise relative error is
# undefined at zeros); lse: max |gpu - ref| / max(1, |ref|).
TOL = {"bf16": dict(t=2e-2, lse=1e-3), "f32": dict(t=1e-4, lse=1e-4)}


def rel_err(got, ref, floor=1e-30):
    """max |got - ref| / max(max |ref|, floor).  `floor` is for cases whose exact result is 0
    (a single visible key has dS = 0): there the error is measured against the size of the
    terms that cancel, which the caller states."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if ref.size == 0:
        return 0.0
    assert np.all(np.isfinite(got)), "non-finite values in the GPU result"
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), floor))


def fro_err(got, ref, floor=1e-30):
    """Second metric: ||got - ref||_F / max(||ref||_F, floor)."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    if ref.size == 0:
        return 0.0
    return float(np.linalg.norm((got - ref).ravel()) / max(np.linalg.norm(ref.ravel()), floor))


def lse_err(got, ref):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    if ref.size == 0:
        return 0.0
    assert np.all(np.isfinite(got)), "non-finite lse"
    return float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max())


class Staged:
    """One tensor in three forms: device tensor (what the kernels read), float64 copy of
    exactly those values (what the oracle reads)."""

    def __init__(self, x_f32: np.ndarray, kind: str, device="cuda"):
        if kind == "bf16":
            bits = synth.f32_to_bf16_bits(x_f32)
            self.f64 = synth.bf16_bits_to_f64(bits).reshape(x_f32.shape)
            self.dev = torch.from_numpy(bits.view(np.int16).reshape(x_f32.shape)).to(device).view(torch.bfloat16)
        else:
            self.f64 = x_f32.astype(np.float64)
            self.dev = torch.from_numpy(np.ascontiguousarray(x_f32)).to(device)


def to_np(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float64).cpu().numpy()


def stage_all(B, l_x, H, d, seed, kind, std=1.0):
    q, k, v, do = synth.make_inputs(B, l_x, H, d, seed, std)
    return tuple(Staged(a, kind) for a in (q, k, v, do))


FwdPlan = collections.namedtuple("FwdPlan", "row_blocks groups splits")
BwdPlan = collections.namedtuple("BwdPlan", "splits groups one_pass own skinny narrow")


def _plan(name, cls, s0, l_s, l_x, B, H, d, causal, *flags):
    plan, i64 = (ctypes.c_int * len(cls._fields))(), ctypes.c_int64
    call = getattr(lss.load(), name)
    lss._check(call(*map(i64, (s0, l_s, l_x, B, H, d)), *(ctypes.c_int(int(f)) for f in (causal, *flags)), plan))
    return cls(*plan)


def fwd_plan(B, l_x, H, d, s0, l_s, causal, drop=False, elem_bytes=2):
    """What a forward call launches (csrc/lss_plan.h)."""
    return _plan("lss_plan_fwd", FwdPlan, s0, l_s, l_x, B, H, d, causal, drop, elem_bytes)


def bwd_plan(B, l_x, H, d, s0, l_s, causal, drop=False, elem_bytes=2, over_out=False):
    """What a backward call launches (csrc/lss_plan.h)."""
    return _plan("lss_plan_bwd", BwdPlan, s0, l_s, l_x, B, H, d, causal, drop, elem_bytes, over_out)


# Tiles of the products (GemmTile of csrc/lss_gemm_plan.h)
TILES = ("256x256", "128x128", "128x128 by two", "128x128 of eight", "64x64", "64x64 in groups", "32x64", "32x32")


def _linear_plan(op, rows, K, N):
    plan, i64 = (ctypes.c_int * 4)(), ctypes.c_int64
    lss._check(lss.load().lss_plan_linear(ctypes.c_int(op), i64(rows), i64(K), i64(N), plan))
    return plan


def _project_plan(op, B, l_x, H, d, l_s, rows_valid):
    plan, i64 = (ctypes.c_int * 8)(), ctypes.c_int64
    lss._check(lss.load().lss_plan_project(ctypes.c_int(op), *map(i64, (l_s, l_x, rows_valid, B, H, d)), plan))
    return plan


def linear_plan(op, rows, K, N):
    """(tile, chunks of rows) of linear_fwd (op 0), linear_bwd_input (1) or linear_bwd_weight (2)."""
    plan = _linear_plan(op, rows, K, N)
    return TILES[plan[0]], plan[1]


def linear_form(op, rows, K, N):
    """(groups of wavefronts that share a contraction, slots of their rings) of the same."""
    return tuple(_linear_plan(op, rows, K, N)[2:4])


def project_plan(op, B, l_x, H, d, l_s, rows_valid):
    """The tile of project_qkv (op 0) or project_bwd (1); tile and chunks of dW_q, tile and chunks of dW_kv (2)."""
    plan = _project_plan(op, B, l_x, H, d, l_s, rows_valid)
    return (TILES[plan[0]], plan[1], TILES[plan[2]], plan[3]) if op == 2 else TILES[plan[0]]


def project_form(op, B, l_x, H, d, l_s, rows_valid):
    """(groups of wavefronts that share a contraction, slots of their rings) of project_qkv (op 0), project_bwd (1) or dW_kv (2)."""
    plan = _project_plan(op, B, l_x, H, d, l_s, rows_valid)
    return tuple(plan[6:8] if op == 2 else plan[1:3])

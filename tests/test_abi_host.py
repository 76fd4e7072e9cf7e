"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before launching anything."""
import ctypes
import re
from pathlib import Path

import pytest

from paper_2311_02382_amd import lss

ROOT = Path(__file__).resolve().parent.parent


@pytest.fixture(scope="module")
def lib():
    if not lss.LIB_PATH.exists():
        from paper_2311_02382_amd.build import build_library
        build_library(verbose=False)
    return lss.load()


def test_every_declared_symbol_is_exported(lib):
    header = (ROOT / "include" / "lss_attn.h").read_text()
    declared = set(re.findall(r"\b(lss_[a-z0-9_]+)\s*\(", header))
    assert declared == set(lss.EXPORTS), declared ^ set(lss.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    assert lib.lss_version() >= 100


def _fwd(lib, q=0x1000, k=0x2000, v=0x3000, s0=0, l_s=128, l_x=256, B=1, H=1, d=64, causal=1, out=0x4000,
         lse=0x5000, f32=False):
    fn = lib.lss_segment_attn_fwd_f32 if f32 else lib.lss_segment_attn_fwd
    return fn(q, k, v, s0, l_s, l_x, B, H, d, causal, out, lse, None)


def test_bad_arguments_are_rejected_without_launching(lib):
    # fake (never dereferenced) device addresses: every call below must fail in the host checks
    assert _fwd(lib, d=32) == -3 and "64 and 128" in lib.lss_last_error().decode()
    assert _fwd(lib, d=96, f32=True) == -3
    assert _fwd(lib, s0=200) == -5            # 200 + 128 > 256
    assert _fwd(lib, s0=-1) == -5
    assert _fwd(lib, l_s=-1) == -2
    assert _fwd(lib, l_x=0, l_s=0) == -2
    assert _fwd(lib, B=70000) == -2
    assert _fwd(lib, q=0) == -1
    assert _fwd(lib, lse=0) == -1
    assert _fwd(lib, k=0x2008) == -4
    assert _fwd(lib, out=0x4004, f32=True) == -4
    # empty calls succeed and touch nothing
    assert _fwd(lib, l_s=0) == 0
    assert _fwd(lib, B=0) == 0


def test_workspace_is_required_and_sized(lib):
    need = lib.lss_workspace_bytes(128, 256, 1, 1, 64, 2)
    assert need > 0
    assert lib.lss_workspace_bytes(128, 256, 1, 1, 32, 2) == 0     # unsupported d
    assert lib.lss_workspace_bytes(128, 256, 1, 1, 64, 3) == 0     # unsupported element size
    assert lib.lss_set_workspace(None, 0) == 0
    assert _fwd(lib) == -6 and "workspace" in lib.lss_last_error().decode()
    assert lib.lss_set_workspace(0x10000, need - 1) == 0
    assert _fwd(lib) == -6
    assert lib.lss_set_workspace(0x10008, need) == -4
    assert lib.lss_set_workspace(None, 64) == -1
    assert lib.lss_set_workspace(None, 0) == 0
    # room for half the bytes of 16 splits' partial outputs is enough, a byte less is not
    need = lib.lss_workspace_bytes(128, 8192, 1, 1, 64, 2)
    assert lib.lss_set_workspace(0x10000, need - 16 * 128 * 64 * 2 - 1) == 0
    assert _fwd(lib, l_x=8192) == -6
    assert lib.lss_set_workspace(None, 0) == 0
    # a skinny segment needs room for its split partial results
    assert lib.lss_workspace_bytes(128, 8192, 1, 1, 64, 2) > 4 * 128 * 64 * 4


def test_backward_and_reduce_argument_checks(lib):
    bwd = lib.lss_segment_attn_bwd
    a = dict(q=0x1000, k=0x2000, v=0x3000, out=0x4000, lse=0x5000, dO=0x6000, dq=0x7000, dk=0x8000, dv=0x9000)

    def call(s0=0, l_s=128, l_x=256, B=1, H=1, d=64, **kw):
        p = dict(a, **kw)
        return bwd(p["q"], p["k"], p["v"], s0, l_s, l_x, B, H, d, 1, p["out"], p["lse"], p["dO"], p["dq"],
                   p["dk"], p["dv"], None)

    assert call(d=80) == -3
    assert call(s0=129) == -5
    assert call(dk=0) == -1
    assert call(dO=0) == -1
    assert call(dv=0x9004) == -4
    assert call() == -6        # no workspace set
    red = lib.lss_reduce_partials
    parts = (ctypes.c_void_p * 2)(0x1000, 0x2000)
    assert red(parts, 0, None, 256, 1, 1, 64, 0x3000, None) == -2
    assert red(None, 2, None, 256, 1, 1, 64, 0x3000, None) == -1
    assert red(parts, 2, None, 256, 1, 1, 64, 0, None) == -1
    assert red(parts, 2, None, 256, 1, 1, 64, 0x2000, None) == -5   # out aliases parts[1]
    bad = (ctypes.c_void_p * 2)(0x1000, 0x2004)
    assert red(bad, 2, None, 256, 1, 1, 64, 0x3000, None) == -4
    nul = (ctypes.c_void_p * 2)(0x1000, None)
    assert red(nul, 2, None, 256, 1, 1, 64, 0x3000, None) == -1


def test_per_call_flags_and_workspace(lib):
    # the general forms: unknown flag bits, a caller's own workspace (size, alignment) -- all host checks
    need = lib.lss_workspace_bytes(128, 256, 1, 1, 64, 2)
    f = lib.lss_segment_attn_fwd_ex
    g = lib.lss_segment_attn_bwd_ex

    def fwd(flags=0, ws=0x10000, nbytes=need, eb=2):
        return f(0x1000, 0x2000, 0x3000, 0, 128, 256, 1, 1, 64, 1, 0.0, 0, eb, flags, ws, nbytes, 0x4000, 0x5000, None)

    def bwd(flags=1, ws=0x10000, nbytes=need, eb=2, p=0.0):
        return g(0x1000, 0x2000, 0x3000, 0, 128, 256, 1, 1, 64, 1, p, 0, eb, flags, ws, nbytes, 0x4000, 0x5000, 0x6000,
                 0x7000, 0x8000, 0x9000, None)

    assert fwd(flags=2) == -5 and b"flag" in lib.lss_last_error()
    assert bwd(flags=6) == -5
    assert fwd(nbytes=need - 1) == -6 and b"passed" in lib.lss_last_error()
    assert bwd(nbytes=need - 1) == -6
    assert fwd(ws=0x10004) == -4
    assert fwd(eb=3) == -2
    assert bwd(p=1.0) == -5
    assert lib.lss_set_workspace(None, 0) == 0
    assert fwd(ws=None, nbytes=0) == -6 and b"registered" in lib.lss_last_error()
    pb = lib.lss_project_bwd_ex
    assert pb(0x1000, 0x2000, 0x3000, 0x4000, 0x5000, 128, 256, 256, 1, 2, 64, 8, 0x6000, 0x7000, None) == -5


def test_projection_weight_gradient_argument_checks(lib):
    f = lib.lss_project_bwd_weight

    def g(x=0x1000, dq=0x2000, dk=0x3000, dv=0x4000, s0=0, l_s=128, l_x=256, rv=256, B=1, H=2, d=64, dwq=0x5000, dwkv=0x6000,
          scratch=0x7000, nbytes=1 << 30):
        return f(x, dq, dk, dv, s0, l_s, l_x, rv, B, H, d, dwq, dwkv, scratch, nbytes, None)

    assert g(H=1) == -2 and g(d=32) == -3 and g(s0=200) == -5
    assert g(rv=257) == -5 and g(rv=-1) == -5
    assert g(dwq=0) == -1 and g(x=0) == -1 and g(dk=0) == -1 and g(dq=0) == -1
    assert g(dv=0x4004) == -4
    need = lib.lss_project_bwd_weight_scratch_bytes(4096, 24576, 4, 16, 64)
    assert need == 4 * 4 * 1024 * 2048 * 4
    assert g(l_s=4096, l_x=24576, rv=24576, B=4, H=16, scratch=0, nbytes=0) == -6
    assert g(l_s=4096, l_x=24576, rv=24576, B=4, H=16, nbytes=need - 1) == -6
    assert lib.lss_project_bwd_weight_scratch_bytes(128, 256, 1, 1, 64) == 0     # E_m = 64: unsupported


def test_layer_operation_argument_checks(lib):
    pe = lib.lss_embed_pe_fwd

    def f(tok=0x1000, table=0x2000, s0=0, l_s=128, l_x=256, B=1, E=64, x=0x3000):
        return pe(tok, table, s0, l_s, l_x, B, E, x, None)

    assert f(E=12) == -2 and f(E=0) == -2 and f(l_x=0) == -2 and f(l_s=-1) == -2
    assert f(s0=129) == -5 and f(s0=-1) == -5
    assert f(tok=0) == -1 and f(x=0) == -1 and f(table=0x2004) == -4
    assert f(B=0) == 0 and f(l_s=0) == 0
    assert lib.lss_embed_pe_bwd(0x1000, 128, 2, 12, 0x2000, None) == -2
    assert lib.lss_embed_pe_bwd(0x1000, 128, 2, 64, None, None) == -1
    assert lib.lss_embed_pe_bwd(None, 0, 2, 64, None, None) == 0

    ra = lib.lss_residual_dropout_add
    assert ra(0x1000, 0x2000, 0, 16, 2, 60, 0.1, 5, 0x3000, None) == -2
    assert ra(0x1000, 0x2000, -1, 16, 2, 64, 0.1, 5, 0x3000, None) == -5
    assert ra(0x1000, 0x2000, 0, 16, 2, 64, 1.0, 5, 0x3000, None) == -5
    assert ra(0x1000, None, 0, 16, 2, 64, 0.1, 5, 0x3000, None) == -1
    assert ra(0x1004, 0x2000, 0, 16, 2, 64, 0.1, 5, 0x3000, None) == -4
    assert ra(None, None, 0, 0, 2, 64, 0.1, 5, None, None) == 0
    ln = lib.lss_layernorm_fwd
    assert ln(0x1000, 0x2000, 0x3000, 1e-5, 4, 4104, 0x4000, 0x5000, 0x6000, None) == -2      # wider than 4096
    assert b"4096" in lib.lss_last_error()
    assert ln(0x1000, 0x2000, 0x3000, 1e-5, 4, 60, 0x4000, 0x5000, 0x6000, None) == -2
    assert ln(0x1000, 0x2000, 0x3000, -1.0, 4, 64, 0x4000, 0x5000, 0x6000, None) == -5
    assert ln(0x1000, None, 0x3000, 1e-5, 4, 64, 0x4000, 0x5000, 0x6000, None) == -1
    assert ln(0x1000, 0x2000, 0x3000, 1e-5, 0, 64, 0x4000, 0x5000, 0x6000, None) == 0
    assert lib.lss_layernorm_bwd_scratch_bytes(33, 512) == 2 * 2 * 512 * 4
    assert lib.lss_layernorm_bwd_scratch_bytes(0, 512) == 0
    lb = lib.lss_layernorm_bwd
    assert lb(0x1000, 0x2000, 0x3000, 0x4000, 0x5000, 33, 512, 0x6000, 0x7000, 0x8000, 0x9000, 8191, None) == -6
    assert lb(0x1000, 0x2000, 0x3000, 0x4000, 0x5000, 33, 512, 0x6000, 0x7000, 0x8000, None, 0, None) == -6
    assert lb(0x1000, 0x2000, 0x3000, 0x4000, 0x5000, 33, 512, 0x6000, None, 0x8000, 0x9000, 8192, None) == -1

    for fn in (lib.lss_linear_fwd, lib.lss_linear_bwd_input):
        assert fn(0x1000, 0x2000, 16, 192, 256, 0x3000, None) == -2      # K not a multiple of 128
        assert fn(0x1000, 0x2000, 16, 256, 64, 0x3000, None) == -2
        assert fn(0x1000, 0x2000, -1, 256, 256, 0x3000, None) == -2
        assert fn(0x1000, 0x2000, 2 ** 31, 256, 256, 0x3000, None) == -2
        assert fn(0x1000, 0, 16, 256, 256, 0x3000, None) == -1
        assert fn(0x1008, 0x2000, 16, 256, 256, 0x3000, None) == -4
        assert fn(0, 0, 0, 256, 256, 0, None) == 0
    wg = lib.lss_linear_bwd_weight
    assert lib.lss_linear_bwd_weight_scratch_bytes(64, 128, 128) == 0               # one chunk: written in place
    assert lib.lss_linear_bwd_weight_scratch_bytes(5000, 128, 128) == 10 * 128 * 128 * 4
    assert lib.lss_linear_bwd_weight_scratch_bytes(5000, 100, 128) == 0
    assert wg(0x1000, 0x2000, 64, 128, 192, 0x3000, None, 0, None) == -2
    assert wg(0x1000, 0x2000, 64, 128, 128, None, None, 0, None) == -1
    assert wg(None, 0x2000, 64, 128, 128, 0x3000, None, 0, None) == -1
    assert wg(0x1000, 0x2008, 64, 128, 128, 0x3000, None, 0, None) == -4
    assert wg(0x1000, 0x2000, 5000, 128, 128, 0x3000, None, 0, None) == -6
    assert wg(0x1000, 0x2000, 5000, 128, 128, 0x3000, 0x4000, 10 * 128 * 128 * 4 - 1, None) == -6
    assert lib.lss_linear_gelu_fwd(0x1000, 0x2000, 16, 256, 256, 0x3000, None, None) == -1
    assert lib.lss_linear_gelu_fwd(0x1000, 0x2000, 16, 256, 256, 0x3000, 0x4008, None) == -4
    assert lib.lss_linear_gelu_fwd(0x1000, 0x2000, 16, 256, 200, 0x3000, 0x4000, None) == -2
    assert lib.lss_linear_bwd_input_gelu(0x1000, 0x2000, None, 16, 256, 256, 0x3000, None) == -1
    assert lib.lss_linear_bwd_input_gelu(0x1000, 0x2000, 0x4004, 16, 256, 256, 0x3000, None) == -4
    assert lib.lss_linear_bwd_input_gelu(None, None, None, 0, 256, 256, None, None) == 0
    assert lib.lss_gelu_fwd(0x1000, 12, 0x2000, None) == -2
    assert lib.lss_gelu_fwd(0x1000, 16, None, None) == -1
    assert lib.lss_gelu_bwd(0x1000, 0x2000, 16, 0x3004, None) == -4
    assert lib.lss_gelu_bwd(None, None, 0, None, None) == 0


def test_projection_argument_checks(lib):
    fwd, bwd = lib.lss_project_qkv, lib.lss_project_bwd

    def f(x=0x1000, wq=0x2000, wkv=0x3000, s0=0, l_s=128, l_x=256, B=1, H=2, d=64, q=0x4000, k=0x5000, v=0x6000):
        return fwd(x, wq, wkv, s0, l_s, l_x, B, H, d, q, k, v, None)

    assert f(H=1) == -2 and b"multiple of 128" in lib.lss_last_error()     # E_m = 64
    assert f(H=3) == -2                                                     # E_m = 192
    assert f(d=32) == -3
    assert f(s0=200) == -5
    assert f(x=0) == -1 and f(wkv=0) == -1 and f(q=0) == -1
    assert f(k=0x5008) == -4
    assert f(B=0) == 0
    assert f(l_s=0, q=0, B=0) == 0

    def g(dq=0x1000, dk=0x2000, dv=0x3000, wq=0x4000, wkv=0x5000, l_s=128, l_x=256, rv=256, B=1, H=2, d=64,
          dxq=0x6000, dxp=0x7000):
        return bwd(dq, dk, dv, wq, wkv, l_s, l_x, rv, B, H, d, dxq, dxp, None)

    assert g(H=1) == -2
    assert g(rv=257) == -5 and g(rv=-1) == -5
    assert g(dk=0) == -1 and g(dxp=0) == -1 and g(dq=0) == -1
    assert g(dv=0x3004) == -4
    assert g(B=0) == 0


def test_dropout_argument_checks(lib):
    fwd, bwd = lib.lss_segment_attn_fwd_dropout, lib.lss_segment_attn_bwd_dropout

    def f(p=0.1, eb=2, d=64, s0=0):
        return fwd(0x1000, 0x2000, 0x3000, s0, 128, 256, 1, 1, d, 1, p, 7, eb, 0x4000, 0x5000, None)

    assert f(p=1.0) == -5 and b"dropout" in lib.lss_last_error()
    assert f(p=-0.5) == -5
    assert f(p=float("nan")) == -5
    assert f(eb=3) == -2
    assert f(d=32) == -3
    assert f(s0=200) == -5
    assert f() == -6            # arguments fine: stops at the missing workspace
    assert f(eb=4) == -6
    assert bwd(0x1000, 0x2000, 0x3000, 0, 128, 256, 1, 1, 64, 1, 1.5, 7, 2, 0x4000, 0x5000, 0x6000, 0x7000,
               0x8000, 0x9000, None) == -5
    assert bwd(0x1000, 0x2000, 0x3000, 0, 128, 256, 1, 1, 64, 1, 0.5, 7, 2, 0x4000, 0x5000, 0x6000, 0x7000,
               0x8000, 0x9000, None) == -6


def test_every_kernel_is_timed_under_its_own_name(lib):
    # names as a profiler prints them: each __global__ function of the library has an id, each id names such a function, and
    # the benchmark knows every attention kernel
    import sys
    sys.path.insert(0, str(ROOT))
    import bench
    from paper_2311_02382_amd import timing
    source = "".join(p.read_text() for p in (ROOT / "paper_2311_02382_amd" / "csrc").glob("*.hip") if "microbench" not in p.name)
    kernels = set(re.findall(r"__global__[^;{]*?\bvoid (\w+)\(", source)) | set(re.findall(r"\) void (\w+_kernel)\(", source))
    named = {n.split(":")[0] for n in timing.kernel_names().values()}
    assert kernels and named == kernels, named ^ kernels
    attention = {k for k in kernels if k.startswith(("fwd_", "bwd_"))}
    assert attention == set(bench.FWD_KERNELS) | set(bench.BWD_KERNELS)
    assert set(bench.ALGO_PRODUCTS) == set(bench.EXEC_PRODUCTS) == attention - {"fwd_merge_kernel", "bwd_dq_merge_kernel", "bwd_prep_bf16_kernel", "bwd_rowdot_kernel"}


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    # no library, no result: the binding has no other path to fall back on
    monkeypatch.setattr(lss, "_lib", None)
    monkeypatch.setattr(lss, "LIB_PATH", tmp_path / "liblss_attn.so")
    with pytest.raises(RuntimeError, match="no fallback"):
        lss.load()
    with pytest.raises(RuntimeError):
        lss.lss_version()


def test_binding_refuses_another_torch_and_another_python(lib, monkeypatch):
    # its native half takes tensors as C++ objects: only the torch it was built for, and a file name for this Python alone
    import importlib.machinery
    from paper_2311_02382_amd import _lss_torch
    assert _lss_torch.__file__.endswith(importlib.machinery.EXTENSION_SUFFIXES[0]) and "cpython" in importlib.machinery.EXTENSION_SUFFIXES[0]
    monkeypatch.setattr(lss, "_native", None)
    assert lss._bind() is _lss_torch
    monkeypatch.setattr(lss, "_native", None)
    monkeypatch.setattr(lss.torch, "__version__", "1.0.0")
    with pytest.raises(RuntimeError, match="built for torch .* and this is torch 1.0.0"):
        lss.lss_gelu_fwd(None)
    monkeypatch.setitem(__import__("sys").modules, "paper_2311_02382_amd._lss_torch", None)
    monkeypatch.delattr("paper_2311_02382_amd._lss_torch")
    with pytest.raises(RuntimeError, match="no fallback"):
        lss.lss_gelu_fwd(None)


def test_product_package_does_not_touch_the_oracle():
    # the oracle is test infrastructure: nothing under the package imports it
    pkg = ROOT / "paper_2311_02382_amd"
    for path in pkg.rglob("*.py"):
        text = path.read_text()
        assert "import oracle" not in text and "from oracle" not in text, path
    for path in (pkg / "csrc").iterdir():
        assert "oracle" not in path.read_text().lower(), path


def test_bench_refuses_more_than_one_gpu():
    # one GPU's share of the path: no collectives, no second GPU -- said before anything touches a device
    import subprocess
    import sys
    root = Path(__file__).resolve().parents[1]
    r = subprocess.run([sys.executable, str(root / "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "--gpus 2 is not supported" in r.stderr and r.stdout == ""

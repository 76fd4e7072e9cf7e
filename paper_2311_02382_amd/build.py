"""Builds liblss_attn.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2311_02382_amd.build                # the library and the binding's native half
    python -m paper_2311_02382_amd.build --microbench   # also lss_microbench (issue-rate microbenchmarks, a stand-alone program)

hipcc cross-compiles without a GPU.  The library lands next to this file so that it
travels with the source tree; nothing is installed.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
INCLUDE = PKG.parent / "include"
LIB = PKG / "liblss_attn.so"
OBJ_DIR = PKG / "_build"

SOURCES = ["lss_fwd.hip", "lss_fwd_bf16.hip", "lss_bwd.hip", "lss_bwd_bf16.hip", "lss_f32.hip", "lss_reduce.hip", "lss_proj.hip", "lss_rows.hip", "lss_timing.hip", "lss_api.hip"]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-instruction results stay in ordinary VGPRs (the softmax reads them with vector ALU
    # ops); accumulation-only registers may still be placed in the AGPR half
    "-mllvm", "-amdgpu-mfma-vgpr-form",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> Path:
    obj = OBJ_DIR / (Path(src).stem + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", "-c", str(CSRC / src), "-o", str(obj)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def binding_path() -> Path:
    """The native half of the binding; the name carries the Python ABI, so another Python does not load it."""
    import sysconfig
    return PKG / f"_lss_torch{sysconfig.get_config_var('EXT_SUFFIX')}"


def _compile_binding() -> Path:
    """csrc/lss_torch.cpp (host code only, against the installed torch's headers)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    obj = OBJ_DIR / "lss_torch.o"
    include = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], "/opt/rocm/include", str(INCLUDE)]
    # the torch and HIP headers are written for either vendor: these two macros name this one
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DLSS_TORCH_VERSION="{torch.__version__}"',
           *(x for d in include for x in ("-isystem", d)), "-c", str(CSRC / "lss_torch.cpp"), "-o", str(obj)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on lss_torch.cpp:\n{r.stderr}")
    return obj


def _link_binding(obj: Path) -> None:
    import torch
    out = binding_path()
    tmp = out.with_suffix(f".so.tmp{os.getpid()}")
    libs = Path(torch.__file__).parent / "lib"
    cmd = ["g++", "-shared", "-o", str(tmp), str(obj), f"-L{PKG}", "-l:liblss_attn.so", f"-L{libs}", "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link of the binding failed:\n{r.stderr}")
    os.replace(tmp, out)
    (PKG / "_lss_torch.so").unlink(missing_ok=True)       # a former name


def build_library(verbose: bool = True) -> Path:
    """Compile every HIP source and link liblss_attn.so, then the binding's native half.  Always recompiles."""
    OBJ_DIR.mkdir(exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as pool:
        binding = pool.submit(_compile_binding)
        objs = list(pool.map(_compile, SOURCES))
        binding_obj = binding.result()
    tmp = LIB.with_suffix(f".so.tmp{os.getpid()}")
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(tmp), *map(str, objs)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    _link_binding(binding_obj)
    if verbose:
        print(f"built {LIB} ({LIB.stat().st_size} bytes)")
    return LIB


MICROBENCH = PKG / "lss_microbench"


def build_microbench(verbose: bool = True) -> Path:
    """Compile csrc/lss_microbench.hip into the stand-alone program lss_microbench."""
    cmd = [_hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-mllvm", "-amdgpu-mfma-vgpr-form", str(CSRC / "lss_microbench.hip"), "-o", str(MICROBENCH)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on lss_microbench.hip:\n{r.stderr}")
    if verbose:
        print(f"built {MICROBENCH}")
    return MICROBENCH


if __name__ == "__main__":
    build_library()
    if "--microbench" in sys.argv[1:]:
        build_microbench()
    sys.exit(0)

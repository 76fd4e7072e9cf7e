"""Rules that host and device code share, driven by small host programs under the undefined-behaviour sanitizer (CPU)."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent


def _run(tmp_path, name, *flags):
    exe = tmp_path / name
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", *flags, f"-I{ROOT}/paper_2311_02382_amd/csrc", "-o", str(exe),
                    str(ROOT / "tests" / "host" / f"{name}.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "clean" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]


def test_every_work_item_belongs_to_one_workgroup(tmp_path):
    _run(tmp_path, "grid_check")


def test_kernel_limits_are_set_on_every_gpu_of_the_process(tmp_path):
    _run(tmp_path, "device_once_check", "-pthread")


def test_backward_plan_counts_the_launches_that_are_made(tmp_path):
    _run(tmp_path, "plan_check")


def test_forward_plan_takes_a_short_one_of_the_measured_forms(tmp_path):
    _run(tmp_path, "fwd_plan_check")


def test_no_launcher_keeps_a_limit_per_process():
    # HIP keeps a kernel's limits per GPU: they are raised through DeviceOnce only
    csrc = ROOT / "paper_2311_02382_amd" / "csrc"
    sets = [p.name for p in csrc.iterdir() if "hipFuncSetAttribute" in p.read_text()]
    assert sets == ["lss_kernels.h"]

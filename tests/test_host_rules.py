"""Rules that host and device code share, driven by small host programs under the undefined-behaviour sanitizer (CPU)."""
import re
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


def test_product_plan_takes_a_tile_there_is_a_kernel_for(tmp_path):
    _run(tmp_path, "gemm_plan_check")


def test_layernorm_backward_takes_one_launch_where_it_is_shorter(tmp_path):
    _run(tmp_path, "rows_plan_check")


def test_results_of_large_products_are_stored_past_the_caches(tmp_path):
    # Two stores that differ in the non-temporal hint only are one plain store to the compiler's middle end: what counts is the
    # generated code.  Every kernel of the projection GEMM has both kinds.
    from paper_2311_02382_amd import build
    out = tmp_path / "proj.s"
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, f"-I{build.INCLUDE}", f"-I{build.CSRC}", "-S", "--offload-device-only", str(build.CSRC / "lss_proj.hip"),
                    "-o", str(out)], check=True, capture_output=True, timeout=300)
    bodies = re.findall(r"^(_Z\w*proj_gemm_kernel\w+):(.*?)s_endpgm\n", out.read_text(), re.S | re.M)
    assert len(bodies) == 25
    for name, body in bodies:
        past = len(re.findall(r"global_store_dwordx4.*\bnt\b", body))
        assert past > 0 and past <= len(re.findall(r"global_store_dwordx4", body)) - past, name


def test_no_launcher_keeps_a_limit_per_process():
    # HIP keeps a kernel's limits per GPU: they are raised through DeviceOnce only
    csrc = ROOT / "paper_2311_02382_amd" / "csrc"
    sets = [p.name for p in csrc.iterdir() if "hipFuncSetAttribute" in p.read_text()]
    assert sets == ["lss_kernels.h"]


def test_assembly_matrix_instructions_have_their_wait_states(tmp_path):
    # The products' wide tiles issue their matrix instructions as assembly, whose operands the compiler's hazard recognizer does not look at: no vector
    # instruction may write an operand (copies of accumulators around a loop, of fragments ahead of their use) within two wait states, and the
    # accumulators are read behind the wait at the end only.
    from paper_2311_02382_amd import build
    out = tmp_path / "proj.s"
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, f"-I{build.INCLUDE}", f"-I{build.CSRC}", "-S", "--offload-device-only", str(build.CSRC / "lss_proj.hip"),
                    "-o", str(out)], check=True, capture_output=True, timeout=300)

    def registers(operand):
        m = re.fullmatch(r"([av])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
        if not m:
            return set()
        first, last = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
        return {(m[1], i) for i in range(first, last + 1)}

    bodies = re.findall(r"^(_Z\w*gemm_kernel\w*GemmWide\w+):(.*?)\.Lfunc_end", out.read_text(), re.S | re.M)
    assert bodies
    for name, body in bodies:
        code = [re.sub(r";.*", "", line).strip() for line in body.splitlines() if re.match(r"\t[a-z]", line)]
        products = 0
        for i, line in enumerate(code):
            if not line.startswith("v_mfma"):
                continue
            products += 1
            used = set().union(*(registers(x) for x in line.split(None, 1)[1].split(",")))
            states = 0
            for before in reversed(code[max(i - 2, 0):i]):
                if states >= 2:
                    break
                op = before.split()[0]
                if op.startswith("v_") and not op.startswith("v_mfma"):
                    assert not registers(before.split(None, 1)[1].split(",")[0]) & used, (name, before, line)
                states += int(before.split()[1]) + 1 if op == "s_nop" else 1
        # (read as soon as none is a matrix instruction's any more)
        for i, line in enumerate(code):
            if line.startswith("v_accvgpr_read") and any(x.startswith("v_mfma") for x in code[max(i - 8, 0):i]):
                assert "s_nop 15" in code[max(i - 8, 0):i], (name, line)
        assert products >= 96 and code.count("s_nop 15") >= 2, name

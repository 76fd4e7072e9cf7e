"""What the compiler made of the kernels: their assembly, and which instructions may run within a number of wait states ahead of another."""
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor


def assembly(directory, sources):
    """{source: assembly of its kernels}, with the flags of the build"""
    from paper_2311_02382_amd import build

    def one(source):
        out = directory / f"{source}.s"
        subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, f"-I{build.INCLUDE}", f"-I{build.CSRC}", "-S", "--offload-device-only", str(build.CSRC / source),
                        "-o", str(out)], check=True, capture_output=True, timeout=600)
        return out.read_text()

    with ThreadPoolExecutor(max_workers=6) as pool:
        return dict(zip(sources, pool.map(one, sources)))


def kernels(text):
    """{name: lines} of the kernels in an assembly text, each with its labels and instructions only"""
    found = {}
    for name, body in re.findall(r"^(_Z\w+):(.*?)^\.Lfunc_end", text, re.S | re.M):
        lines = (re.sub(r";.*", "", line).strip() for line in body.splitlines())
        found[name] = [line for line in lines if line and (line.endswith(":") or not line.startswith("."))]
    return found


def registers(operand):
    """{(kind, number)} of one operand: v, a and s registers, vcc as a pair of its own"""
    operand = operand.strip().strip("|-")
    if operand == "vcc":
        return {("vcc", 0)}
    m = re.fullmatch(r"([avs])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    first, last = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], i) for i in range(first, last + 1)}


def operands(line):
    parts = line.split(None, 1)
    return [registers(x.split()[0] if x.split() else "") for x in parts[1].split(",")] if len(parts) > 1 else []


def written(line):
    """what a vector instruction writes"""
    op, regs = line.split()[0], operands(line)
    out = set(regs[0]) if regs else set()
    if len(regs) > 1 and ("_co_" in op or op.startswith(("v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32", "v_swap", "v_permlane"))):
        out |= regs[1]
    return out


class Flow:
    """Instructions of a kernel and the ones that may run right before each"""

    def __init__(self, lines):
        self.code, labels, pending = [], {}, []
        for line in lines:
            if line.endswith(":"):
                pending.append(line[:-1])
            else:
                for label in pending:
                    labels[label] = len(self.code)
                pending = []
                self.code.append(line)
        self.before = [[] for _ in self.code]
        for i, line in enumerate(self.code):
            op = line.split()[0]
            if i + 1 < len(self.code) and op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                self.before[i + 1].append(i)
            if op == "s_branch" or op.startswith("s_cbranch"):
                target = labels.get(line.split()[1])
                if target is not None:
                    self.before[target].append(i)

    def within(self, i, states):
        """every instruction fewer than `states` wait states ahead of instruction i, along any path"""
        best, todo = {}, [(p, 0) for p in self.before[i]]
        while todo:
            at, waited = todo.pop()
            if waited >= states or best.get(at, states) <= waited:
                continue
            best[at] = waited
            line = self.code[at]
            waited += int(line.split()[1]) + 1 if line.startswith("s_nop") else 1
            todo += [(p, waited) for p in self.before[at]]
        return [(self.code[at], waited) for at, waited in best.items()]

"""Builds libpolykv.so (HIP, gfx950 only) in-tree with hipcc.  `python -m paper_2604_24971_amd.build`."""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpolykv.so")
SOURCES = ["polykv_api.hip", "polykv_codec.hip", "polykv_attend.hip", "polykv_attend_mfma.hip"]
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed-fp32 VALU forms stay off on these machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return r.stdout


def _check_no_scratch(remarks: str):
    """The matrix-core attention kernel keeps its accumulators, parked query operands and score tiles in all 512
    registers of a wave; builds in which the register allocator spilled part of that to scratch memory returned
    wrong results on the GPU.  Refuse such a build: every instantiation must come out without scratch."""
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "ScratchSize" in line and name and "attend_mfma_" in name:
            size = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
            if size and not os.environ.get("POLYKV_BUILD_ALLOW_SCRATCH"):   # (the variable is for timing experiments only)
                raise RuntimeError("%s spills %d bytes per lane to scratch: reduce its register use" % (name, size))


def _registers(text: str):
    out = set()
    for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        if m.group(1):
            out.update((m.group(1), k) for k in range(int(m.group(2)), int(m.group(3)) + 1))
        else:
            out.add((m.group(4), int(m.group(5))))
    return out


# Wait states after a vector write before a matrix instruction or a DPP source reads the register, and after a matrix
# instruction before a vector (or memory) access to its result.
_OPERAND_WAIT, _RESULT_WAIT = 2, 12


class _WaitStates:
    """What is still under way at a place in the code: the registers that vector instructions and matrix instructions have
    written, and the wait states since."""

    def __init__(self, name, writes=None, results=None):
        self.name, self.writes, self.results = name, dict(writes or {}), list(results or [])

    def copy(self):
        return _WaitStates(self.name, self.writes, self.results)

    def clear(self):
        self.writes, self.results = {}, []

    def busy(self):
        return bool(self.writes or self.results)

    def _fresh(self, regs):
        return any(self.writes.get(r, _OPERAND_WAIT) < _OPERAND_WAIT for r in regs)

    def _unfinished(self, regs):
        return any(regs & result for result, _ in self.results)

    def step(self, op, rest, text):
        mfma = "mfma_f32_32x32x16" in op    # (the smaller ones are all the compiler's own)
        vector = op.startswith("v_")
        if self.busy() or mfma or vector:
            operands = [_registers(o) for o in rest.split(",")]
            if mfma:
                if any(self._fresh(o) for o in operands[1:]):
                    raise RuntimeError("%s: operand written too shortly before: %s" % (self.name, text))
                if self._unfinished(operands[1] | operands[2]):
                    raise RuntimeError("%s: result of a matrix instruction read too early: %s" % (self.name, text))
            elif vector or op.startswith(("ds_", "buffer_", "global_", "scratch_", "flat_")):
                if self.results and self._unfinished(set().union(*operands)):
                    raise RuntimeError("%s: result of a matrix instruction accessed too early: %s" % (self.name, text))
                if "_dpp" in op and self._fresh(operands[1]):
                    raise RuntimeError("%s: DPP source written too shortly before: %s" % (self.name, text))
        states = int(rest) + 1 if op == "s_nop" else 1
        if self.writes:
            self.writes = {r: n + states for r, n in self.writes.items() if n + states < _OPERAND_WAIT}
        if self.results:
            self.results = [(regs, n + states) for regs, n in self.results if n + states < _RESULT_WAIT]
        if mfma:
            self.results.append((operands[0], 0))
        elif vector and not op.startswith("v_cmp"):
            for o in operands[:2] if "swap" in op else operands[:1]:
                self.writes.update((r, 0) for r in o)


def _check_wait_states(asm_path):
    """Part of the attention kernel's matrix and DPP instructions are inline assembly, whose wait states the compiler does not
    keep: two between a vector write of an operand (DPP: of the first source) and the instruction that reads it, twelve
    between a matrix instruction and a vector (or memory) access to its result.  The source is laid out so that they are
    kept; what the register allocator inserts in between is not under its control.  Refuse a build in which a distance is
    too short, along the text or across a branch.  Returns the number of matrix instructions that were checked."""
    name, code, labels, matrix = None, [], {}, 0

    def follow(at, state):      # from a branch's target, as long as something is under way
        while at < len(code) and state.busy():
            op, rest, text = code[at]
            state.step(op, rest, text)
            if op.startswith(("s_branch", "s_cbranch")) and rest in labels and state.busy():
                follow(labels[rest], state.copy())
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                return
            at += 1

    def check_function():
        state = _WaitStates(name)
        for op, rest, text in code:
            state.step(op, rest, text)
            if op.startswith(("s_branch", "s_cbranch")) and rest in labels and state.busy():
                follow(labels[rest], state.copy())
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                state.clear()

    for line in open(asm_path):
        m = re.match(r"^([\w.$]+):", line)
        if m and m.group(1).startswith("_Z"):
            check_function()
            name, code, labels = m.group(1), [], {}
        elif m:
            labels[m.group(1)] = len(code)
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.replace("\t", " ").partition(" ")
        matrix += "mfma_f32_32x32x16" in op
        code.append((op, rest.strip(), text))
    check_function()
    if not matrix:
        raise RuntimeError("%s holds no matrix instruction: the check reads the wrong file" % asm_path)
    return matrix


def build_library(verbose: bool = True, extra_flags=()) -> str:
    """Compile every source and link the shared library; always recompiles."""
    hipcc = _hipcc()
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, s.replace(".hip", ".o")) for s in SOURCES]

    def compile_one(i):
        cmd = [hipcc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, SOURCES[i]), "-o", objs[i]]
        if SOURCES[i] == "polykv_attend_mfma.hip":
            log = _run(cmd + ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics", "-save-temps=obj"])
            _check_no_scratch(log)
            _check_wait_states(os.path.join(objdir, "polykv_attend_mfma-hip-amdgcn-amd-amdhsa-gfx950.s"))
            return "\n".join(l for l in log.splitlines() if "kernel-resource-usage" not in l)
        return _run(cmd)

    with ThreadPoolExecutor(max_workers=4) as ex:
        logs = list(ex.map(compile_one, range(len(SOURCES))))
    logs.append(_run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB]))
    if verbose:
        for log in logs:
            if log.strip():
                print(log, file=sys.stderr)
        print("built", LIB, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build_library()

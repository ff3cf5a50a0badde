"""Builds librelax_mi355.so for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librelax_mi355.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC] + os.environ.get("RELAX_EXTRA_HIPCC_FLAGS", "").split()


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


# Sources whose kernels stream from HBM with their working set in registers: a variant that the register allocator
# spills to scratch memory still computes the right values, several times slower (measured: 4 x on a one-row matvec), so
# the build refuses it.  {source: substring of the mangled kernel names it applies to}
NO_SCRATCH = {"gemv_q4_reg.hip": "gemv_q4_reg_kernel", "gemv_reg_f16.hip": "gemv_q4_reg_kernel", "gemv_reg_q3.hip": "gemv_q4_reg_kernel", "gemv_q4_long.hip": "gemv_q4_long_kernel",
              "gemv_q3.hip": "gemv_q3", "fewrow_q4g32.hip": "fewrow_kernel", "fewrow_q4g64.hip": "fewrow_kernel",
              "fewrow_q4g128.hip": "fewrow_kernel", "fewrow_q3.hip": "fewrow_kernel", "fewrow_f16.hip": "fewrow_kernel", "attn_decode.hip": "attn_"}
REMARK = "-Rpass-analysis=kernel-resource-usage"


def scratch_users(remarks: str, name_part: str):
    """(kernel, bytes per lane) of every kernel in the compiler's resource-usage remarks that uses scratch memory."""
    bad, name = [], None
    for line in remarks.splitlines():
        if "remark: Function Name:" in line:
            name = line.split("Function Name:")[1].split("[")[0].strip()
        elif "ScratchSize [bytes/lane]:" in line and name is not None:
            size = int(line.split("ScratchSize [bytes/lane]:")[1].split("[")[0])
            if size > 0 and name_part in name:
                bad.append((name, size))
    return bad


# Sources that write their MFMAs as inline asm (accumulators in place): the compiler does not see to the distances the matrix
# instructions need there, so the build checks them in the assembly.
MFMA_ASM = "gemm_packed_"
OPERAND_SLOTS = 2        # issue slots between a vector operation and an MFMA that reads what it wrote
RESULT_SLOTS = 18        # ... and between an MFMA and another instruction that touches its result


def _registers(operand: str):
    """The vector and accumulation registers of an operand, whatever modifiers stand around it."""
    m = re.search(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))(?!\w)", operand.split()[0] if operand.split() else "")
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[3])) if m[2] else (int(m[4]), int(m[4]))
    return {(m[1], i) for i in range(lo, hi + 1)}


class _Instruction:
    def __init__(self, text: str):
        self.text = text
        self.name, _, rest = text.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        regs = [_registers(o) for o in ops]
        self.touched = set().union(*regs)
        self.mfma = self.name.startswith("v_mfma")
        self.written = (regs[0] | regs[1] if self.name.startswith("v_swap") else regs[0]) if self.name.startswith("v_") else set()
        self.slots = int(ops[0], 0) + 1 if self.name == "s_nop" else 1
        self.target = ops[0] if self.name.startswith(("s_branch", "s_cbranch")) else None
        self.falls_through = self.name not in ("s_branch", "s_endpgm")


def _listing(assembly: str):
    """(instructions, {label: index of the instruction behind it}) of an assembly listing."""
    code, labels = [], {}
    for line in assembly.splitlines():
        text = line.split(";")[0].strip()
        if text.endswith(":"):
            labels[text[:-1]] = len(code)
        elif text and not text.startswith("."):
            code.append(_Instruction(text))
    return code, labels


def mfma_hazards(assembly: str):
    """Instructions of an assembly listing that come too soon behind or in front of an MFMA on some path, loops' back edges among them, as texts."""
    code, labels = _listing(assembly)
    bad = []
    for i, first in enumerate(code):
        if not first.mfma and not first.written:
            continue
        limit = RESULT_SLOTS if first.mfma else OPERAND_SLOTS
        todo = [(i, 0)]                                      # (instruction, issue slots from the first one to it)
        while todo:
            at, slots = todo.pop()
            ins = code[at]
            if at != i or slots:
                if first.mfma:
                    hit = not ins.mfma and first.written & ins.touched
                else:
                    hit = ins.mfma and first.written & ins.touched
                if hit:
                    bad.append("%s -> %s" % (first.text, ins.text))
                slots += ins.slots
            if slots >= limit:
                continue
            slots = max(slots, 0)
            if ins.falls_through and at + 1 < len(code):
                todo.append((at + 1, slots))
            if ins.target in labels and labels[ins.target] < len(code):
                todo.append((labels[ins.target], slots))
    return bad


def mfma_loop_scratch(assembly: str):
    """Accesses to scratch memory inside loops that hold MFMAs, as texts."""
    code, labels = _listing(assembly)
    bad = []
    for i, ins in enumerate(code):
        if ins.target in labels and labels[ins.target] <= i:
            loop = code[labels[ins.target]:i + 1]
            if any(x.mfma for x in loop):
                bad += [x.text for x in loop if x.name.startswith("scratch_")]
    return bad


def check_mfma_listing(src: str, assembly: str) -> None:
    if "v_mfma" not in assembly:
        raise RuntimeError("%s: no MFMA in the assembly listing" % src)
    bad = mfma_hazards(assembly)
    if bad:
        raise RuntimeError("%s: instructions too close to an MFMA: %s" % (src, "; ".join(bad[:8])))
    bad = mfma_loop_scratch(assembly)
    if bad:
        raise RuntimeError("%s: scratch memory in a loop of MFMAs: %s" % (src, "; ".join(bad[:8])))


def _check_mfma_asm(src: str, folder: str) -> None:
    listings = [f for f in os.listdir(folder) if f.endswith("gfx950.s")]
    if len(listings) != 1:
        raise RuntimeError("%s: no assembly listing to check (%s)" % (src, ", ".join(listings)))
    with open(os.path.join(folder, listings[0])) as f:
        check_mfma_listing(src, f.read())


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src[:-4] + ".o")
    guarded = src in NO_SCRATCH
    cmd = [HIPCC] + FLAGS + ([REMARK] if guarded else [])
    with tempfile.TemporaryDirectory() as folder:            # of the intermediate files where the assembly is checked
        checked = src.startswith(MFMA_ASM)
        kept = os.path.join(folder, os.path.basename(obj)) if checked else obj
        res = subprocess.run(cmd + (["--save-temps=obj"] if checked else []) + ["-c", os.path.join(CSRC, src), "-o", kept], capture_output=True, text=True)
        if checked and res.returncode == 0:
            _check_mfma_asm(src, folder)
            shutil.move(kept, obj)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, res.stdout, res.stderr))
    if guarded:
        bad = scratch_users(res.stderr, NO_SCRATCH[src])
        if bad:
            raise RuntimeError("%s: kernels that spill to scratch memory: %s" % (src, ", ".join("%s (%d B/lane)" % b for b in bad)))
        res.stderr = "\n".join(l for l in res.stderr.splitlines() if REMARK not in l and not l.lstrip().startswith(("|", "^", "In file included from")) and
                               not (l.strip()[:1].isdigit() and "|" in l))
    warn = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(sources()))) as pool:
        objs = list(pool.map(_compile, sources()))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()

"""Build-time checks of the compiled gfx950 code: no matrix instruction under a narrowed execution mask, no accumulator register
touched before the matrix instruction that writes it has (scan_agpr_reads).

`v_mfma_*` ignores EXEC.  A source-level `if (cond) acc = mfma(...)` whose condition lives in a vector
register is compiled to an execution-mask region (`s_and_saveexec_b64` ... `s_or_b64 exec`); the compiler
normally jumps over the region when no lane is left (`s_cbranch_execz`), but drops that jump when the region is
short and holds nothing it considers unsafe to run with an empty mask, and MFMA is not on that list.  The
region's MFMAs then run although the condition is false for the whole wavefront.  The kernels avoid this by
deriving every condition that guards an MFMA from scalars (`__builtin_amdgcn_readfirstlane` of the wavefront
index), which gives scalar branches; this module checks the result on the emitted assembly.

    python -m paper_2603_25702_amd.isa_lint          # compiles csrc/*.hip to assembly and scans it
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor
from typing import List, Tuple

from .build import CSRC, FLAGS, SOURCES, _hipcc

_NARROW = re.compile(r"^s_(and|andn2|or|xor|nand|nor|xnor|orn2)_saveexec_b64\b")
_EXEC_WRITE = re.compile(r"^s_(and|andn2|xor|mov)_b64\s+exec\b")
_EXEC_RESTORE = re.compile(r"^s_or_b64\s+exec\b")
_KERNEL = re.compile(r"^(_Z\w+):")


def scan_asm(text: str) -> List[Tuple[str, int, str]]:
    """Returns (kernel, line number, instruction) for every MFMA that follows a narrowing of EXEC with no
    `s_cbranch_execz` in between, up to the point where EXEC is widened again or control leaves the block."""
    kernel, narrowed, guarded = "?", False, False
    found = []
    for no, raw in enumerate(text.splitlines(), 1):
        m = _KERNEL.match(raw)
        if m:
            kernel, narrowed = m.group(1), False
        ins = raw.split(";")[0].strip()
        if not ins or ins.startswith("."):
            continue
        if _NARROW.match(ins) or _EXEC_WRITE.match(ins):
            narrowed, guarded = True, False
        elif _EXEC_RESTORE.match(ins) or ins.startswith(("s_branch", "s_endpgm")):
            narrowed = False
        elif ins.startswith("s_cbranch_execz") and narrowed:
            guarded = True
        elif ins.startswith(("v_mfma", "v_smfmac")) and narrowed and not guarded:
            found.append((kernel, no, ins))
    return found


_AREG = re.compile(r"(?<![\w.])a(?:\[(\d+):(\d+)\]|(\d+))(?!\w)")
_LABEL = re.compile(r"^([.\w$]+):")
MFMA_RESULT_WAIT = 11   # wait states between a 16x16x32 product and whatever else touches its result (the compiler gives its own eight)


def _aregs(operand: str) -> range:
    m = _AREG.search(operand)
    return range(0) if not m else range(int(m.group(3)), int(m.group(3)) + 1) if m.group(3) else range(int(m.group(1)), int(m.group(2)) + 1)


def _basic_blocks(lines):
    """(instructions, successors) of a kernel's basic blocks."""
    blocks, at = [[]], {}
    for no, ins, asm in lines:
        m = _LABEL.match(ins)
        if m:
            if blocks[-1]:
                blocks.append([])
            at[m.group(1)] = len(blocks) - 1
            continue
        blocks[-1].append((no, ins, asm))
        if ins.startswith(("s_branch", "s_cbranch", "s_endpgm", "s_setpc")):
            blocks.append([])
    out = []
    for i, block in enumerate(blocks):
        last = block[-1][1] if block else ""
        to = [at[t] for t in last.split()[1:2] if last.startswith(("s_branch", "s_cbranch")) and t in at]
        if not last.startswith(("s_branch", "s_endpgm", "s_setpc")) and i + 1 < len(blocks):
            to.append(i + 1)
        out.append((block, to))
    return out


def _pass_block(block, pending, found=None):
    """Wait states that accumulator registers still need behind a block, from those they need in front of it."""
    now, ready = 0, dict(pending)   # register -> time at which its result is there
    for no, ins, asm in block:
        name, _, rest = ins.partition(" ")
        operands = rest.split(",")
        touched = operands[1:3] if name.startswith("v_mfma") else operands   # (products wait for the accumulators of one another by themselves)
        if found is not None and any(ready.get(reg, 0) > now for operand in touched for reg in _aregs(operand)):
            found.append((no, ins))
        nop = re.match(r"^s_nop\s+(\d+)", ins)
        now += int(nop.group(1)) + 1 if nop else 1
        if asm and name.startswith("v_mfma_f32_16x16x32"):
            for reg in _aregs(operands[0]):
                ready[reg] = now + MFMA_RESULT_WAIT
    return {reg: t - now for reg, t in ready.items() if t > now}


def scan_agpr_reads(text: str) -> List[Tuple[str, int, str]]:
    """Returns (kernel, line number, instruction) for every instruction that touches an accumulator register too soon behind an
    MFMA of inline assembly that writes it, on any path: a copy, a store or a spill of it, another value for it, an MFMA with it as A or
    B.  (The compiler does not know what these instructions are and waits for none of them.)"""
    kernels, lines, asm = [], [], False
    for no, raw in enumerate(text.splitlines(), 1):
        m = _KERNEL.match(raw)
        asm = "#ASMSTART" in raw or (asm and "#ASMEND" not in raw)
        ins = raw.split(";")[0].strip()
        if m:
            lines = []
            kernels.append((m.group(1), lines))
        elif kernels and ins and (not ins.startswith(".") or ins.endswith(":")):
            lines.append((no, ins, asm))
    found = []
    for kernel, lines in kernels:
        if not any(asm and ins.startswith("v_mfma_f32_16x16x32") for _, ins, asm in lines):
            continue
        blocks = _basic_blocks(lines)
        start = [{} for _ in blocks]     # longest waits on any way there
        work = list(range(len(blocks)))
        while work:
            i = work.pop()
            behind = _pass_block(blocks[i][0], start[i])
            for j in blocks[i][1]:
                more = {reg: w for reg, w in behind.items() if w > start[j].get(reg, 0)}
                if more:
                    start[j].update(more)
                    work.append(j)
        for (block, _), pending in zip(blocks, start):
            here = []
            _pass_block(block, pending, here)
            found += [(kernel, no, ins) for no, ins in here]
    return found


def compile_to_asm(src: str, out_dir: str) -> str:
    out = os.path.join(out_dir, src.replace(".hip", ".s"))
    flags = [f for f in FLAGS if f != "-fPIC"]
    cmd = [_hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc -S failed on {src}:\n{r.stderr}")
    return out


def lint_sources(sources=None, jobs: int = 6) -> List[Tuple[str, str, int, str]]:
    sources = [s for s in (sources or SOURCES)
               if "mfma" in open(os.path.join(CSRC, s)).read() or s in ("attention.hip", "attention_wide.hip")]
    with tempfile.TemporaryDirectory() as tmp:
        with ThreadPoolExecutor(max_workers=jobs) as ex:
            paths = list(ex.map(lambda s: compile_to_asm(s, tmp), sources))
        found = []
        for src, path in zip(sources, paths):
            text = open(path).read()
            found += [(src, k, no, ins) for k, no, ins in scan_asm(text) + scan_agpr_reads(text)]
    return found


if __name__ == "__main__":
    bad = lint_sources()
    for src, k, no, ins in bad:
        print(f"{src}: {k}: line {no}: {ins}")
    print(f"{len(bad)} matrix instruction(s) under a narrowed execution mask without a skip branch, or results touched too early")
    sys.exit(1 if bad else 0)

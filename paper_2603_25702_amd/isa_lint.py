"""Build-time check of the compiled gfx950 code: no matrix instruction under a narrowed execution mask.

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


_MFMA_AGPR = re.compile(r"^v_mfma_f32_16x16x32\w*\s+a\[(\d+):(\d+)\]")
_AGPR_READ = re.compile(r"^(?:v_accvgpr_(?:read_b32|mov_b32)\s+\w+,\s*a(\d+)|ds_write\w*\s+.*\ba\[?(\d+))")
MFMA_RESULT_WAIT = 11   # wait states between a product of eight passes and a vector instruction that reads it


def scan_agpr_reads(text: str) -> List[Tuple[str, int, str]]:
    """Returns (kernel, line number, instruction) for every read of an accumulator register too soon behind the MFMA that
    writes it, in program order."""
    kernel, now, written = "?", 0, {}
    found = []
    for no, raw in enumerate(text.splitlines(), 1):
        m = _KERNEL.match(raw)
        if m:
            kernel, now, written = m.group(1), 0, {}
        ins = raw.split(";")[0].strip()
        if not ins or ins.startswith(".") or ins.endswith(":"):
            continue
        m = _AGPR_READ.match(ins)
        if m:
            reg = int(m.group(1) or m.group(2))
            if now - written.get(reg, -10 ** 9) < MFMA_RESULT_WAIT:
                found.append((kernel, no, ins))
        m = re.match(r"^v_accvgpr_(?:write_b32|mov_b32)\s+a(\d+)", ins)
        if m:
            written.pop(int(m.group(1)), None)   # another value
        nop = re.match(r"^s_nop\s+(\d+)", ins)
        now += int(nop.group(1)) + 1 if nop else 1
        m = _MFMA_AGPR.match(ins)
        if m:
            for reg in range(int(m.group(1)), int(m.group(2)) + 1):
                written[reg] = now
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
    print(f"{len(bad)} matrix instruction(s) under a narrowed execution mask without a skip branch, or results read too early")
    sys.exit(1 if bad else 0)

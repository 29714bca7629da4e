"""The grid sweeps' published face records: stores of 16 bytes, whose data
registers the next vector instructions must not overwrite for two wait states
(a store of more than 64 bits reads them that late).  The compiler keeps that
distance for stores that it sees, so no such store may be inline assembly; in
the library as it is built, no vector instruction next to one writes its data."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1701_05913_amd", "libkrylov.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _statements(text):
    """The asm statements' strings."""
    return re.findall(r"\basm\b[^(]*\(\s*((?:\"[^\"]*\"\s*)+)", text)


def test_no_wide_store_in_inline_assembly():
    found = []
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_1701_05913_amd", "csrc", "*"))):
        with open(path) as f:
            found += [(os.path.basename(path), s) for s in _statements(f.read())
                      if re.search(r"(global|flat|buffer)_store_dwordx[34]", s)]
    assert not found, found


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$|v(\d+)$", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def test_no_published_data_overwritten_too_soon(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(OBJDUMP):
        pytest.skip("no built library or no disassembler")
    shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", "libkrylov.so"], cwd=tmp_path, check=True, capture_output=True)
    stores, bad = 0, []
    for path in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", str(path)], check=True, capture_output=True, text=True).stdout
        lines = [ln.split("//")[0].strip() for ln in text.splitlines()]
        for at, ln in enumerate(lines):
            m = re.match(r"(global|buffer)_store_dwordx4 (.*)\bsc1\b", ln)
            if not m:
                continue
            stores += 1
            ops = [o.strip() for o in m.group(2).split(",")]
            data = _registers(ops[0] if m.group(1) == "buffer" else ops[1])
            states = 0
            for nxt in lines[at + 1:at + 3]:
                if nxt.startswith("v_") and states < 2:
                    if _registers(nxt.split(None, 1)[1].split(",")[0].strip()) & data:
                        bad.append((path.name, ln, nxt))
                nop = re.match(r"s_nop (\d+)", nxt)
                states += int(nop.group(1)) + 1 if nop else 1
    assert stores > 0, "no published store found"
    assert not bad, bad[:3]

"""The grid sweeps' published face records in the library as it is built: an
inline-assembly store of 16 bytes, whose data registers the next vector
instructions must not overwrite for two wait states (a store of more than 64
bits reads them that late).  The compiler does not see such a store, so every
one has to be followed by its own wait states."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1701_05913_amd", "libkrylov.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _code_objects(folder):
    shutil.copy(LIB, folder)
    subprocess.run([OBJDUMP, "--offloading", "libkrylov.so"], cwd=folder, check=True, capture_output=True)
    return [os.path.join(folder, f) for f in sorted(os.listdir(folder)) if f.endswith("gfx950")]


def test_wait_states_follow_every_published_store(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(OBJDUMP):
        pytest.skip("no built library or no disassembler")
    stores, bad = 0, []
    for path in _code_objects(str(tmp_path)):
        text = subprocess.run([OBJDUMP, "-d", path], check=True, capture_output=True, text=True).stdout
        if "sc1" not in text:
            continue
        lines = [ln.split("//")[0].strip() for ln in text.splitlines()]
        for at, ln in enumerate(lines):
            if re.match(r"global_store_dwordx[34] .*\bsc1\b", ln):
                stores += 1
                after = re.match(r"s_nop (\d+)", lines[at + 1])
                if not after or int(after.group(1)) < 1:
                    bad.append((os.path.basename(path), ln, lines[at + 1]))
    assert stores > 0, "no published store found"
    assert not bad, bad[:3]

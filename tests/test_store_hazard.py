"""The built kernels keep a 16-byte buffer store and a vector instruction that
overwrites its data two wait states apart: closer, the store was seen to read
the new value.  Checked on the disassembly of the library's own code."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2312_00229_amd import _lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)$", operand)
    return {int(m[1])} if m else set()


def hazards(lines):
    found = []
    for i, line in enumerate(lines):
        if not re.match(r"buffer_store_dwordx[34] ", line):
            continue
        data = _registers(line.split(None, 1)[1].split(", ")[0])
        waited = 0
        for nxt in lines[i + 1:i + 3]:
            op = nxt.split()[0]
            if op == "s_nop":
                waited += int(nxt.split()[1])
            elif op.startswith("v_") and not op.startswith("v_cmp") and waited < 2:
                if _registers(nxt.split(None, 1)[1].split(", ")[0]) & data:
                    found.append((line, nxt))
            waited += 1
    return found


def test_scan_finds_a_planted_hazard():
    store = "buffer_store_dwordx4 v[8:11], v36, s[12:15], s38 offen"
    write = "v_mul_f32_e32 v10, s43, v23"
    assert hazards([store, write, "s_nop 0"])
    assert hazards([store, "s_add_i32 s0, s0, 1", write])
    assert not hazards([store, "s_nop 1", write])
    assert not hazards([store, "v_mul_f32_e32 v12, s43, v23", "s_nop 0"])


def test_no_store_data_hazard_in_the_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(os.path.join(os.path.dirname(_lib.__file__), "libweno_zoom.so"), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    objects = sorted(p for p in tmp_path.iterdir() if "gfx950" in p.name)
    assert objects
    stores = 0
    for obj in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True,
                              text=True).stdout
        lines = [ln.split("//")[0].strip() for ln in text.splitlines() if ln.startswith("\t")]
        stores += sum(ln.startswith("buffer_store_dwordx4") for ln in lines)
        assert not hazards(lines), (obj.name, hazards(lines)[:3])
    assert stores > 0

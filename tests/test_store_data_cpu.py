"""The built kernels leave a store's data registers alone until the store has read them.

A vector-memory store of more than 64 bits reads its data registers after it has
issued: on gfx950 a VALU instruction may write them only two issue slots later.  The
compiler keeps that distance except for buffer stores with a register as scalar
offset, where it assumes that none is needed; such stores have ended up with the
low word of a double replaced by the value computed next.  This reads the
AMD assembly of the library built here and finds no store with its data overwritten
within two slots, whatever its form."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1909_02894_amd", "libdirac.so")
OBJDUMP = "/opt/rocm/lib/llvm/bin/llvm-objdump"
SLOTS = 2
STORE = re.compile(r"(buffer|global|flat|scratch)_store_dwordx[34]\b")
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(operand):
    out = set()
    for f, lo, hi, one in REG.findall(operand):
        out |= {(f, i) for i in range(int(lo or one), int(hi or one) + 1)}
    return out


def overwritten_store_data(lines):
    """(function, store, overwriting instruction, slots between) of every offending store."""
    found, stores, func, pending = [], 0, "", []
    for line in lines:
        text = line.split("//")[0].strip()
        if not line.startswith((" ", "\t")) or not text:
            m = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", text)
            func, pending = (m.group(1) if m else func), []
            continue
        op, _, rest = text.partition(" ")
        ops = rest.split(",")
        if pending and op.startswith("v_"):
            written = registers(ops[0]) | (registers(ops[1]) if "swap" in op else set())
            found += [(func, s, text, d) for s, data, d in pending if written & data]
        step = int(ops[0], 0) + 1 if op == "s_nop" else 1
        pending = [(s, data, d + step) for s, data, d in pending if d + step < SLOTS]
        if op in ("s_endpgm", "s_branch", "s_setpc_b64"):
            pending = []
        if STORE.match(op):
            stores += 1
            pending.append((text, registers(ops[0] if op.startswith("buffer") else ops[1]), 0))
    return found, stores


def test_the_scan_finds_a_planted_overwrite():
    store = "\tbuffer_store_dwordx4 v[64:67], v130, s[0:3], s6 offen sc1 // 0"
    assert overwritten_store_data([store, "\tv_mov_b32_e32 v64, v52 // 4"])[0]
    assert overwritten_store_data([store, "\ts_nop 0", "\tv_permlane32_swap_b32_e32 v1, v67"])[0]
    assert not overwritten_store_data([store, "\ts_nop 1", "\tv_mov_b32_e32 v64, v52"])[0]
    assert not overwritten_store_data([store, "\tv_mov_b32_e32 v68, v64", "\tv_mov_b32_e32 v69, v1"])[0]
    assert overwritten_store_data(["\tglobal_store_dwordx4 v0, v[4:7], s[0:1]", "\tv_add_f32 v5, v1, v2"])[0]


@pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(LIB)), reason="needs the built library and llvm-objdump")
def test_no_store_data_is_overwritten_early(tmp_path):
    shutil.copy(LIB, tmp_path / "libdirac.so")
    subprocess.run([OBJDUMP, "--offloading", "libdirac.so"], cwd=tmp_path, check=True, capture_output=True)
    objs = sorted(f for f in os.listdir(tmp_path) if "gfx950" in f)
    assert objs

    def scan(f):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True,
                           text=True)
        return overwritten_store_data(r.stdout.splitlines())

    with ThreadPoolExecutor(4) as ex:
        results = list(ex.map(scan, objs))
    assert sum(n for _, n in results) > 1000
    bad = [b for found, _ in results for b in found]
    assert not bad, (len(bad), bad[:4])

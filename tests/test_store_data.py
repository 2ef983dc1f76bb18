"""The built kernels' machine code: no store of more than 8 bytes is followed
directly by a vector instruction that writes its data registers.  The store
reads them after it has issued; gfx950 needs a wait state between the two
whether the store's scalar offset is a constant (where the compiler keeps it)
or a register (where it does not)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_39816_amd", "libfm.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
WIDE = re.compile(r"(buffer|global|flat|scratch)_store_(dwordx[34]|b96|b128)\b")


def vregs(tok):
    m = re.match(r"v\[(\d+):(\d+)\]$", tok) or re.match(r"v(\d+)$", tok)
    return set(range(int(m[1]), int(m[m.lastindex]) + 1)) if m else set()


def overwritten(text):
    """(kernel, store, next instruction) of every such pair, and the number
    of wide stores."""
    out, stores, fn, prev = [], 0, None, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            fn, prev = m[1], None
            continue
        s = line.split("//")[0].strip()
        if not line.startswith("\t") or not s:
            continue
        if prev and s.startswith("v_"):
            dst = s.split(None, 1)[1].split(",")[0].strip()
            if vregs(dst) & prev[1]:
                out.append((fn, prev[0], s))
        prev = None
        if WIDE.match(s):
            stores += 1
            ops = [t.strip() for t in s.split(None, 1)[1].split(",")]
            prev = (s, vregs(ops[0] if s.startswith("buffer") else ops[1]))
    return out, stores


def test_the_search_finds_such_a_pair():
    pair = ("0000000000000000 <k>:\n\tbuffer_store_dwordx4 v[66:69], v74, s[16:19], s58 offen nt // 00\n"
            "\t{} // 01\n")
    assert overwritten(pair.format("v_fma_f32 v66, s8, v2, 0"))[0]
    assert overwritten(pair.format("v_lshl_add_u64 v[68:69], v[2:3], 0, s[2:3]"))[0]
    assert not overwritten(pair.format("v_fma_f32 v70, s8, v2, 0"))[0]
    assert not overwritten(pair.format("s_nop 0"))[0]


def test_no_store_data_is_overwritten_at_once(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs llvm-objdump")
    if not os.path.exists(LIB):
        pytest.skip("needs the built library")
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objs = glob.glob(str(tmp_path / "*gfx950*"))
    assert objs, "no gfx950 code in the library"
    bad, stores = [], 0
    for o in objs:
        text = subprocess.run([OBJDUMP, "-d", o], check=True, capture_output=True, text=True).stdout
        b, n = overwritten(text)
        bad += b
        stores += n
    assert stores > 0
    assert not bad, bad[:4]

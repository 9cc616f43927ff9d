"""The built device code never overwrites the data of a wide store in the next instruction.

A store of more than 64 bits still reads its data registers after it has issued, so one
other instruction has to follow before a vector instruction writes them.  The compiler
keeps that rule except for buffer stores whose scalar offset is in a register, where it
takes the hardware to need no wait; stored values were the overwriting ones there now and
then (one element of a vector, in some lanes).  Here the library's own code is
disassembled and searched for such pairs, on the CPU."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1912_02165_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump") or "") if os.path.exists(p)), None)


def code_objects(path):
    """The gfx950 code objects bundled in a library."""
    blob = open(path, "rb").read()
    out, at = [], blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                out.append(blob[at + off:at + off + size])
        at = blob.find(MAGIC, p)
    return out


def registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m[1])} if m else set()


def overwritten_stores(text):
    """(wide stores, [(kernel, store, next instruction), ...]) of a disassembly."""
    stores, found, kernel, wide = 0, [], "", None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            kernel, wide = m[1], None
            continue
        line = line.split("//")[0].strip()
        if not line:
            continue
        op, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if wide and op.startswith("v_") and registers(ops[0]) & wide[0]:
            found.append((kernel, wide[1], line))
        wide = None
        if re.fullmatch(r"buffer_store_dwordx[34]", op):
            wide = (registers(ops[0].split()[0]), line)
        elif re.fullmatch(r"(global|flat|scratch)_store_dwordx[34]", op):
            wide = (registers(ops[1].split()[0]), line)
        stores += wide is not None
    return stores, found


def test_search_finds_the_pair():
    """The search itself, on a listing with one such pair among harmless ones."""
    text = """0000 <k>:
    buffer_store_dwordx4 v[4:7], v1, s[0:3], s4 offen sc1  // 0
    s_nop 0
    v_mov_b32_e32 v5, v9
    buffer_store_dwordx4 v[4:7], v1, s[0:3], s4 offen
    v_mov_b32_e32 v8, v4
    buffer_store_dwordx2 v[4:5], v1, s[0:3], s4 offen
    v_mov_b32_e32 v4, v9
    global_store_dwordx4 v[0:1], v[4:7], off
    v_add_f32_e32 v6, v2, v3
"""
    stores, found = overwritten_stores(text)
    assert stores == 3 and [f[2] for f in found] == ["v_add_f32_e32 v6, v2, v3"]


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_no_store_data_overwritten(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    objects = code_objects(build.LIB)
    assert objects, "no gfx950 code in the library"
    total, bad = 0, []
    for i, obj in enumerate(objects):
        f = tmp_path / f"{i}.co"
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", str(f)], capture_output=True, text=True, check=True).stdout
        stores, found = overwritten_stores(text)
        total += stores
        bad += found
    print(f"{len(objects)} code objects, {total} wide stores")
    assert total > 500
    assert not bad, f"{len(bad)} of {total}: {bad[:4]}"

"""The built kernels leave the data of 96- and 128-bit stores alone until the store has read it.

A wide store reads its data registers for a few cycles after it is issued.  The compiler keeps the
next two cycles' instructions from writing them, but not where a buffer store has a scalar offset
register, and on gfx950 such a store needs it as well: it stored what the next instruction wrote.
So no wide store may have a scalar offset register, and none may be followed within two cycles by an
instruction that writes its data.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1312_3265_amd import build

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_images(path):
    """The gfx950 code objects bundled in the library (one per source file)."""
    data = open(path, "rb").read()
    images, pos = [], data.find(MAGIC)
    while pos >= 0:
        (n,) = struct.unpack_from("<Q", data, pos + len(MAGIC))
        q = pos + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, q)
            target = data[q + 24:q + 24 + tlen]
            q += 24 + tlen
            if b"gfx950" in target and size:
                images.append(data[pos + off:pos + off + size])
        pos = data.find(MAGIC, pos + len(MAGIC))
    return images


def _registers(operand):
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo = int(m[2] if m[2] else m[3])
    return {(m[1], k) for k in range(lo, int(m[2] if m[2] else m[4]) + 1)}


def wide_store_faults(text):
    """(wide stores, messages) of a disassembly: scalar offsets, and data written within two
    cycles of the store."""
    stores, faults, function, recent = 0, [], "", []
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            function, recent = m[1], []
            continue
        ins = line.split("//")[0].strip()
        op, _, rest = ins.partition(" ")
        operands = [x.strip() for x in rest.split(",")]
        if op.startswith("v_"):
            written = _registers(operands[0])
            faults += [f"{function}: {s} then {ins}" for s, data, _ in recent if data & written]
        cycles = int(operands[0], 0) + 1 if op == "s_nop" else 1
        recent = [(s, d, age + cycles) for s, d, age in recent if age + cycles < 2]
        if re.match(r"(buffer|global|flat|scratch)_store_dwordx[34]$", op):
            stores += 1
            buf = op.startswith("buffer")
            recent.append((ins, _registers(operands[0 if buf else 1]), 0))
            if buf and re.match(r"s\d|m0", operands[3]):
                faults.append(f"{function}: scalar offset in {ins}")
    return stores, faults


def test_the_scan_finds_both_forms():
    text = """0000000000001000 <kernel>:
        buffer_store_dwordx4 v[26:29], v88, s[48:51], s58 offen // 0
        v_cvt_f64_f32_e32 v[26:27], v22 // 8
        buffer_store_dwordx4 v[2:5], v88, s[48:51], 0 offen // 10
        s_nop 1 // 18
        v_mov_b32_e32 v2, 0 // 1c
        global_store_dwordx4 v[0:1], v[6:9], off // 20
        v_mov_b32_e32 v0, 0 // 28
        v_mov_b32_e32 v9, 0 // 2c"""
    n, faults = wide_store_faults(text)
    assert n == 3 and len(faults) == 3, faults


def test_no_wide_store_loses_its_data():
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs llvm-objdump")
    lib = build.LIB if os.path.exists(build.LIB) else build.build()
    stores, faults = 0, []
    for image in _device_images(lib):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "-"], input=image,
                             capture_output=True, check=True).stdout.decode()
        n, f = wide_store_faults(out)
        stores += n
        faults += f
    assert stores > 1000
    assert not faults, f"{len(faults)} of {stores} wide stores, e.g. {faults[:3]}"

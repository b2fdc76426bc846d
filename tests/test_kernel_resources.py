"""Registers and scratch of the built kernels (CPU only: read from the library's own notes).

A forward kernel that keeps its operands in scratch reloads them for every tile, and each reload
waits for the next stage's loads too: the narrow bf16 form at head dim 64 once spilled 17
registers and ran 24 % slower than the form it replaces.
"""
import os
import re
import struct
import subprocess

import pytest

import paper_2403_04690_amd as na

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_objects(data):
    """The gfx950 code objects of every offload bundle in the library."""
    for m in re.finditer(MAGIC, data):
        at = m.start()
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in triple and size:
                yield data[at + off:at + off + size]


def _spills(tmp_path):
    """(symbol, spilled VGPRs) of every kernel of the library."""
    with open(na.library_path(), "rb") as f:
        data = f.read()
    out = []
    for i, obj in enumerate(_device_objects(data)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for block in notes.split("- .agpr_count")[1:]:
            out.append((re.search(r"\.symbol:\s+(\S+)\.kd", block).group(1),
                        int(re.search(r"\.vgpr_spill_count:\s+(\d+)", block).group(1))))
    return out


def test_forward_kernels_keep_their_operands_in_registers(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    kernels = _spills(tmp_path)
    if not kernels:
        pytest.skip("a library without device code")
    fwd = {s: n for s, n in kernels if "na_fwd_kernel" in s}
    # <rank, D, type, blocks per wave, stage blocks, row form (2: narrow), waves>
    narrow = {s: n for s, n in fwd.items() if re.search(r"Li2ELi\d+ELi2ELi4EEEv", s)}
    assert len(fwd) > 60 and len(narrow) == 16, (len(fwd), len(narrow))
    # up to six values that only the epilogue reads (offsets, row sums); operands take more
    assert {s: n for s, n in fwd.items() if n > 6} == {}
    assert {s: n for s, n in narrow.items() if "DF16b" in s and n} == {}

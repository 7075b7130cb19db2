"""Checks of the device sources and of what the compiler made of them, without
a GPU."""
import glob
import os
import re
import struct
import subprocess

import pytest

from paper_2512_14681_amd import jf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_14681_amd", "csrc")


def asm_statements(text):
    """The text of every asm(...) statement, parentheses matched outside string literals."""
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == "\\" and quoted:
                i += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text[m.start():i]


def test_inline_asm_names_the_m0_it_writes():
    """An asm statement that writes M0 lists it as clobbered: the compiler
    may keep a value of its own there (indexed moves, LDS-DMA builtins,
    messages)."""
    writers = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            for s in asm_statements(f.read()):
                if re.search(r"\bm0\s*,", s):
                    writers.append((os.path.basename(path), s))
    assert writers
    for path, s in writers:
        assert re.search(r':\s*(?:"\w+"\s*,\s*)*"m0"', s), (path, s)


READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel symbol: {vgpr_count, vgpr_spill_count, ...}} of libjf's gfx950 code objects."""
    if not os.path.exists(jf.LIB_PATH) or not os.path.exists(READELF):
        pytest.skip("needs the built library and llvm-readelf")
    with open(jf.LIB_PATH, "rb") as f:
        lib = f.read()
    out, tmp = {}, tmp_path_factory.mktemp("co")
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(magic, lib):
        at = m.start()
        n, = struct.unpack_from("<Q", lib, at + len(magic))
        if not 1 <= n <= 8:
            continue
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, pos)
            ident = lib[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" not in ident:
                continue
            path = tmp / "co.o"
            path.write_bytes(lib[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for block in re.split(r"\n\s+- \.", notes):
                name = re.search(r"\.name:\s+(\S+)", block)
                if name:
                    out[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\b", block)}
    assert out
    return out


def test_attention_keeps_a_chunks_loads_in_flight(kernels):
    """The fp32 form at head_dim 128 of few workgroups loads a chunk's K (2 x
    4 fragments of 8 registers) and V^T (8 x 8) before it computes: with
    fewer than 128 registers some of the loads wait for others (1 row after
    1024 keys 15.4 -> 17.8 us)."""
    name = [k for k in kernels if "k_attnIfLi128ELi1ELb0E" in k]
    assert len(name) == 1
    assert kernels[name[0]]["vgpr_count"] > 128 and kernels[name[0]]["vgpr_spill_count"] == 0

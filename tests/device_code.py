"""The gfx950 code objects inside the built library, as the assembler's tools print them."""

import functools
import os
import re
import shutil
import struct
import subprocess
import tempfile

import paper_2609_34174_amd as gl

_LLVM = "/opt/rocm/llvm/bin"


def tool(name):
    path = shutil.which(name) or os.path.join(_LLVM, name)
    return path if os.path.exists(path) else None


def _code_objects():
    """The gfx950 ELF images of the library's offload bundles (one per source file)."""
    blob = open(gl.LIB_PATH, "rb").read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := blob.find(magic, at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(n if n < 16 else 0):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + idlen]:
                out.append(blob[at + off:at + off + size])
            p += 24 + idlen
        at += len(magic)
    return out


def _each(*cmd):
    for image in _code_objects():
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(image)
            f.flush()
            yield subprocess.run([tool(cmd[0]), *cmd[1:], f.name], capture_output=True, text=True, check=True).stdout


def _names(symbols):
    out = subprocess.run([tool("c++filt")], input="\n".join(symbols), capture_output=True, text=True, check=True).stdout
    return [re.sub(r"\(.*$|^void |gradlev::", "", s) for s in out.splitlines()]


@functools.lru_cache(maxsize=1)
def spills():
    """{kernel: spilled vector registers}"""
    found = {}
    for text in _each("llvm-readelf", "--notes"):
        for block in text.split("- .agpr_count")[1:]:
            name = re.search(r"^\s+\.name:\s+(\S+)", block, re.M)
            found[name[1]] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", block)[1])
    return dict(zip(_names(found), found.values()))


@functools.lru_cache(maxsize=1)
def listing():
    """{kernel: its instructions}"""
    found = {}
    for text in _each("llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr"):
        for part in re.split(r"^<(?=_Z)", text, flags=re.M)[1:]:
            name, body = part.split(">:", 1)
            found[name] = [line.strip() for line in body.splitlines() if line.strip()]
    return dict(zip(_names(found), found.values()))

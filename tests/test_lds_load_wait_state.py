"""Every direct load to LDS in the built library stands at least one instruction behind the last
write of M0, its LDS address: gfx950 needs one wait state between the two, and inline assembly
gets none from the compiler. Read from the library's own gfx950 code."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2201_12854_amd as mca
from paper_2201_12854_amd import build_lib

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _objdump():
    near = os.path.join(os.path.dirname(os.path.realpath(build_lib.hipcc())), "..", "llvm", "bin", "llvm-objdump")
    return shutil.which("llvm-objdump") or next((p for p in (near, "/opt/rocm/llvm/bin/llvm-objdump") if os.path.exists(p)), None)


def _code_objects(path):
    """The gfx950 code objects of a library's offload bundles (magic, count, then per entry its
    offset, size and target name)."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        q = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, q)
            name = data[q + 24:q + 24 + length]
            q += 24 + length
            if build_lib.ARCH.encode() in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def _writes_m0(line):
    op, _, args = line.partition(" ")
    return op.startswith("s_") and args.split(",")[0].strip() == "m0"


def test_m0_wait_state(tmp_path):
    tool = _objdump()
    if tool is None:
        pytest.skip("no llvm-objdump")
    mca.load_library()  # built if it is not there
    loads = 0
    for i, obj in enumerate(_code_objects(build_lib.LIB)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(obj)
        text = subprocess.run([tool, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        kernel, before = "", ""
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if label:
                kernel, before = label.group(1), ""
                continue
            line = line.split("//")[0].strip()
            if not line:
                continue
            if re.match(r"(global_load_lds|buffer_load\w* .*\blds$)", line):
                loads += 1
                assert not _writes_m0(before), (kernel, before, line)
            before = line
    assert loads >= 10  # the streaming passes and the saturated tokens' kernels

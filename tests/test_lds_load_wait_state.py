"""Every direct load to LDS in the built library keeps the wait states that gfx950 asks for and that
inline assembly does not get from the compiler: one behind a write of M0, its LDS address, and five
behind a vector instruction's write of a scalar register that it reads. Read from the library's own
gfx950 code."""
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


def _scalars(operands):
    """The scalar registers named in a list of operands."""
    regs = {"m0"} if re.search(r"\bm0\b", operands) else set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", operands):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(a) for a in re.findall(r"\bs(\d+)\b", operands))
    return regs


def _wait_states(line):
    op, _, arg = line.partition(" ")
    return int(arg) + 1 if op == "s_nop" else 1


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
        kernel, before = "", []
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if label:
                kernel, before = label.group(1), []
                continue
            line = line.split("//")[0].strip()
            if not line:
                continue
            if re.match(r"(global_load_lds|buffer_load\w* .*\blds$)", line):
                loads += 1
                states, reads = 0, _scalars(line) | {"m0"}
                for b in reversed(before):
                    written = _scalars(b.partition(" ")[2].split(",")[0])
                    assert states >= 1 or "m0" not in written, (kernel, b, line)
                    assert not (b.startswith("v_") and written & reads), (kernel, b, line)
                    states += _wait_states(b)
                    if states >= 5:
                        break
            before = before[-8:] + [line]
    assert loads >= 10  # the streaming passes and the saturated tokens' kernels

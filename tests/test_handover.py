"""Kernels whose workgroups hand data to each other inside a launch: every wave's stores have to be done before the barrier behind which
one thread makes them visible to the chip.

That a store is still under way when it should not be shows in no result that a test could force; it can be seen in the machine code of
this library's own build, which is what is read here.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1707_02402_amd", "libdynbatch.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LABEL = "label:"

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs llvm-objdump")


def code_objects(tmp_path):
    """The gfx950 code objects of the library, one per source file: bundle = magic, count, then (offset, size, length of name, name) each."""
    data = open(LIB, "rb").read()
    for i, m in enumerate(re.finditer(MAGIC, data)):
        at = m.start() + len(MAGIC)
        count, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                path = tmp_path / f"object{i}.elf"
                path.write_bytes(data[m.start() + offset:m.start() + offset + size])
                yield str(path)


def kernels(tmp_path, name):
    """{symbol: its instructions, with a LABEL where a branch leads to} of the kernels whose name holds `name`."""
    found = {}
    for path in code_objects(tmp_path):
        table = subprocess.run([OBJDUMP, "-t", path], check=True, capture_output=True, text=True).stdout
        for symbol in sorted({line.split()[-1] for line in table.splitlines() if name in line and " .text" in line and " F " in line}):
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + symbol, path], check=True, capture_output=True, text=True).stdout
            # "instruction // address: encoding <symbol+offset of a branch's target>"
            lines = re.findall(r"^\s+(\S.*?)\s+// ([0-9A-F]+): [0-9A-F ]+(?:<%s(?:\+0x([0-9a-f]+))?>)?$" % re.escape(symbol), text, flags=re.M)
            start = int(lines[0][1], 16)
            targets = {start + int(offset, 16) for _, _, offset in lines if offset}
            found[symbol] = [line for code, address, _ in lines for line in ([LABEL, code] if int(address, 16) in targets else [code])]
    return found


def undone(code):
    """(hand-overs, those of them whose barrier may be reached with stores under way).  A hand-over is a write-back of the L2 and the last barrier before it."""
    total, bad = 0, 0
    for at, line in enumerate(code):
        if not line.startswith("buffer_wbl2"):
            continue
        total += 1
        back = max(i for i in range(at) if code[i].startswith("s_barrier"))
        while True:
            back -= 1
            if re.match(r"s_waitcnt .*vmcnt\(0\)", code[back]):
                break
            if re.match(LABEL + "|s_cbranch|s_branch|global_|buffer_|flat_|scratch_", code[back]):     # other ways here, or something under way
                bad += 1
                break
    return total, bad


@pytest.mark.parametrize("name,variants", [("k_topk_group", 3), ("k_module_persist", 1)])
def test_stores_are_done_before_the_barrier_of_a_handover(tmp_path, name, variants):
    found = kernels(tmp_path, name)
    assert len(found) == variants
    for symbol, code in found.items():
        total, bad = undone(code)
        assert total == 1, symbol
        assert bad == 0, symbol

"""The block loop of the bf16 attention kernel as the built library has it: where
it lies, and the registers of its exponentials' arguments.

The loop's time depends on where its instructions fall in the 32-byte fetches
(1.5 % between the best and the worst of the eight placements), and code before
the loop moves it: the source pads it to 16 bytes past a 32-byte boundary.
The library's own gfx950 code object is disassembled and the loop's first
instruction looked up: the target of the shortest backward branch that spans
all matrix instructions of the kernel.

An exponential's argument (score * scale + offset, the only multiply-adds with a
scalar factor in the loop) is computed in the score's own register. With one
temporary for all of them each would wait for the exponential before it (up to
1 % of a large call).
"""

import os
import re
import struct
import subprocess

import pytest

import paper_2607_16190_amd as fva

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """gfx950 code objects of a library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24 : p + 24 + length].decode()
            p += 24 + length
            if triple.endswith("gfx950") and size:
                yield data[at + off : at + off + size]
        at = data.find(MAGIC, at + 1)


def kernel_code(tmp_path, name):
    """[(address, instruction with its operands, branch target or None)] of the kernel whose mangled name holds `name`."""
    for i, obj in enumerate(code_objects(fva.LIB_PATH)):
        if name.encode() not in obj:
            continue
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout
        m = re.search(r"^([0-9a-f]+) <\w*%s\w*>:\n(.*?)(?:\n\n|\Z)" % name, text, re.S | re.M)
        if not m:
            continue
        base, code = int(m.group(1), 16), []
        for line in m.group(2).split("\n"):
            x = re.match(r"\s+(\S.*?)\s*//\s*([0-9A-F]+):.*?(?:<\w+\+0x([0-9a-f]+)>)?\s*$", line)
            if x:
                code.append((int(x.group(2), 16), x.group(1), base + int(x.group(3), 16) if x.group(3) else None))
        return code
    return None


def block_loop(code):
    """(first, last address) of the block loop."""
    products = [a for a, op, _ in code if "mfma" in op]
    assert len(products) > 100
    loops = [(a - t, t, a) for a, op, t in code
             if t is not None and op.startswith(("s_branch", "s_cbranch")) and t < products[0] and a > products[-1]]
    assert loops
    return min(loops)[1:]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("kernel", ["attn_persistent_kernelILb0E"])
def test_block_loop_starts_16_bytes_past_a_fetch(kernel, tmp_path):
    code = kernel_code(tmp_path, kernel)
    assert code, f"{kernel} not found in {fva.LIB_PATH}"
    assert block_loop(code)[0] % 32 == 16


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("kernel", ["attn_persistent_kernelILb0E"])
def test_exponential_arguments_stay_in_the_scores_registers(kernel, tmp_path):
    code = kernel_code(tmp_path, kernel)
    assert code, f"{kernel} not found in {fva.LIB_PATH}"
    first, last = block_loop(code)
    args = [re.match(r"v_fma_f32 (v\d+), s\d+, (v\d+), v\d+$", op) for a, op, _ in code if first <= a <= last]
    args = [m for m in args if m]
    assert len(args) >= 64  # two halves of 64 keys, 32 scores per lane
    assert all(m.group(1) == m.group(2) for m in args)

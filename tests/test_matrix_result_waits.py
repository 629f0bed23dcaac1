"""The built library's matrix instructions: nothing uses a result too early, and accumulators meet one instruction.

The hardware does not wait for a matrix result: 8 instructions lie between a 16-bit product (16 rows x 16 columns) and the first use of its sums, 10 behind an
fp32 one, unless the use is the next product on the same accumulators (of the same kind here: see the 1D kernels' weighted_sum).  The compiler sees to it; on paths across branches it has
counted wrong, so every path is walked here."""
import collections
import os
import re
import struct
import subprocess

import pytest

from paper_2204_07143_amd.binding import LIB_PATH

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
REGISTER = re.compile(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def wait_of(op):
    assert re.fullmatch(r"v_mfma_f32_16x16x(16|32)_b?f16|v_mfma_f32_16x16x4_f32", op), op
    return 10 if op.endswith("x4_f32") else 8


def registers(text):
    out = set()
    for m in REGISTER.finditer(text):
        out |= {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)} if m[1] else {(m[4], int(m[5]))}
    return out


def code_objects():
    data, at = open(LIB_PATH, "rb").read(), 0
    while (at := data.find(BUNDLE, at)) >= 0:
        count, entry = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + length] and size:
                yield data[at + offset:at + offset + size]
            entry += 24 + length
        at += 24


def kernels(path):
    """(name, [(address, mnemonic, operands)]) of every function of a code object"""
    name, code = None, []
    for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout.splitlines():
        if m := re.match(r"[0-9a-f]+ <(\S+)>:", line):
            if code:
                yield name, code
            name, code = m[1], []
        elif m := re.match(r"\t(\S+)(.*)// ([0-9A-F]+):", line):
            code.append((int(m[3], 16), m[1], m[2].strip()))
    if code:
        yield name, code


def too_early(code):
    at = {c[0]: i for i, c in enumerate(code)}
    for i, (_, op, operands) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        need, result = wait_of(op), registers(operands.split(",")[0])
        reached, todo = {}, [(i + 1, 0)]
        while todo:
            n, waited = todo.pop()
            if n >= len(code) or waited >= need or reached.get(n, need) <= waited:
                continue
            reached[n] = waited
            address, other, rest = code[n]
            if other == "s_endpgm":
                continue
            if other == "s_nop":
                todo.append((n + 1, waited + 1 + int(rest, 0)))
                continue
            if other.startswith(("s_branch", "s_cbranch")):
                if other.startswith("s_cbranch"):
                    todo.append((n + 1, waited + 1))
                offset = int(rest.split(",")[-1])
                todo.append((at[address + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)], waited + 1))
                continue
            if other.startswith("v_mfma"):
                _, a, b, c = (registers(x) for x in rest.split(",")[:4])
                bad = result & (a | b) or (c == result and other != op)
            else:
                bad = result & registers(rest)
            if bad:
                yield f"{op} {operands} -> {other} {rest} after {waited}"
            todo.append((n + 1, waited + 1))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for the library's own code")
def test_no_result_is_used_too_early(tmp_path):
    found, products = collections.defaultdict(list), 0
    for n, data in enumerate(code_objects()):
        path = tmp_path / f"{n}.co"
        path.write_bytes(data)
        for name, code in kernels(str(path)):
            products += sum(c[1].startswith("v_mfma") for c in code)
            found[name] += too_early(code)
    assert products > 5000
    assert not {k: v for k, v in found.items() if v}

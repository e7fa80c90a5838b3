"""Machine code of the persistent 256 x 256 GEMM tile: what its main loop must not contain, and a hazard of instructions written as text."""
import re
import subprocess

import pytest

from test_device_code import LLVM, code_object      # noqa: F401  (fixture)

pytestmark = pytest.mark.skipif(LLVM is None, reason="needs the ROCm LLVM tools")


@pytest.fixture(scope="module")
def kernels(code_object):       # noqa: F811
    """{mangled name: [(address, instruction)]} of the tile's kernels"""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", code_object], check=True, capture_output=True, text=True).stdout
    found, name = {}, None
    for line in text.splitlines():
        label = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if label:
            name = label.group(1)
            continue
        instruction = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if instruction and name and "gemm_tile256" in name:
            found.setdefault(name, []).append((int(instruction.group(2), 16), instruction.group(1)))
    assert len(found) == 12      # five epilogues, the rotation for two head sizes, with and without the strip
    return found


def main_loop(code):
    """The innermost loop that holds the 128 products of a k-tile."""
    at = {address: i for i, (address, _) in enumerate(code)}
    loops = []
    for i, (address, text) in enumerate(code):
        jump = re.match(r"s_c?branch\S*\s+(\d+)", text)
        if jump:
            offset = int(jump.group(1))
            target = address + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)
            if at.get(target, i) < i:
                body = [t for _, t in code[at[target]:i + 1]]
                if sum("v_mfma" in t for t in body) >= 128:
                    loops.append(body)
    return min(loops, key=len)


def test_main_loop(kernels):
    """Nothing but the products, the reads, the copies and the wait for copies: a wait for memory that the compiler adds (for an epilogue's load or
    a reload that it believes in flight) drains the copies once per k-tile, moves between the halves of the register file stand in front of products."""
    for name, code in kernels.items():
        body = main_loop(code)
        assert sum("v_mfma" in t for t in body) in (128, 132, 136), name
        assert not [t for t in body if re.match(r"scratch_|buffer_|v_accvgpr", t)], name
        assert sum("s_waitcnt" in t and "vmcnt" in t for t in body) == 1, name
        assert sum("load_lds" in t for t in body) in (16, 17), name


def scalars(text):
    out = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out |= set(range(int(m.group(1)), int(m.group(2)) + 1)) if m.group(1) else {int(m.group(3))}
    return out


def test_vector_writes_of_scalars(kernels):
    """A scalar register that the vector ALU wrote needs five wait states before a memory instruction reads it; for the copies, which are text, the compiler
    does not keep them."""
    for name, code in kernels.items():
        recent = []      # (registers, wait states, instruction)
        for _, text in code:
            op = text.split()[0]
            if "load_lds" in op:
                age = 0
                for written, states, writer in reversed(recent):
                    if age >= 5:
                        break
                    assert not written & scalars(text), (name, writer, text)
                    age += states
            states = int(text.split()[1], 0) + 1 if op == "s_nop" else 1
            destination = text.split(",")[0]
            if op.startswith("s_") and not re.match(r"s_(nop|cmp|bitcmp|waitcnt|barrier|c?branch)", op):
                recent = [(w - scalars(destination), n, t) for w, n, t in recent]
            vector_write = re.match(r"v_readlane|v_readfirstlane|v_cmp", op)
            recent = (recent + [(scalars(destination) if vector_write else set(), states, text)])[-8:]

"""Machine code of the persistent tiles that compute the whole strip of 16 rows behind a single M-tile, or have fewer than three k-tiles: the rules of the tile
they are made from."""
import re
import subprocess

import pytest

from test_device_code import LLVM, code_object      # noqa: F401  (fixture)
from test_device_code_tile256 import main_loop, test_vector_writes_of_scalars      # noqa: F401  (collected here with this file's kernels)

pytestmark = pytest.mark.skipif(LLVM is None, reason="needs the ROCm LLVM tools")


@pytest.fixture(scope="module")
def kernels(code_object):       # noqa: F811
    """{mangled name: [(address, instruction)]}"""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", code_object], check=True, capture_output=True, text=True).stdout
    found, name = {}, None
    for line in text.splitlines():
        label = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if label:
            name = label.group(1)
            continue
        instruction = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if instruction and name and re.search("gemm_(tile272|short256)", name):
            found.setdefault(name, []).append((int(instruction.group(2), 16), instruction.group(1)))
    assert len(found) == 6 + 12      # five epilogues, the rotation for two head sizes; four epilogues without the strip, with half of it, with the whole
    return found


def test_main_loop(kernels):
    for name, code in kernels.items():
        body = main_loop(code)
        assert sum("v_mfma" in t for t in body) in (128, 132, 136, 144), name      # four of the strip per half, twice that where a V tile swaps the operands
        assert not [t for t in body if re.match(r"scratch_|buffer_|v_accvgpr", t)], name
        assert sum("s_waitcnt" in t and "vmcnt" in t for t in body) == 1, name
        assert sum("load_lds" in t for t in body) in (16, 17), name

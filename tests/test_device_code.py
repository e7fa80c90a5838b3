"""Rules for the gfx950 machine code of the built library that neither the compiler nor a run checks: the instructions of an inline-asm block
get no wait states from the compiler, and results can be right by luck."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = next((d for d in ("/opt/rocm/llvm/bin", "/opt/rocm/lib/llvm/bin") if os.path.exists(os.path.join(d, "llvm-objdump"))), None)
pytestmark = pytest.mark.skipif(LLVM is None, reason="needs the ROCm LLVM tools")


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """The gfx950 code object of the library, unpacked."""
    import paper_2506_05229_amd as P
    if not os.path.exists(P.library_path()):
        from paper_2506_05229_amd.build import build
        build()
    where = tmp_path_factory.mktemp("device_code")
    lib = shutil.copy(P.library_path(), where / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], check=True, capture_output=True, cwd=where)
    found = [f for f in os.listdir(where) if "gfx950" in f]
    assert len(found) == 1, found
    return str(where / found[0])


def test_lds_copies_wait_for_m0(code_object):
    """A scalar write of M0 needs one wait state in front of a global load to LDS."""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", code_object], check=True, capture_output=True, text=True).stdout
    copies, bad, kernel, before = 0, {}, None, ""
    for line in text.splitlines():
        label = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if label:
            kernel, before = label.group(1), ""
            continue
        instruction = line.split("//")[0].strip()
        if not instruction:
            continue
        if "load_lds" in instruction or (instruction.startswith("buffer_load") and re.search(r"\blds\b", instruction)):
            copies += 1
            if re.match(r"s_\w+ m0,", before):
                bad[kernel] = bad.get(kernel, 0) + 1
        before = instruction
    assert copies > 1000          # the pattern still finds the copies
    assert not bad


# Vector registers a kernel may keep in scratch memory (a reload waits behind every copy in flight): the feature-map epilogue of the
# W_Q projection, in the tiles that wide d_mem and large or irregular launches take.
SPILLS = {
    r"gemm_mfma_kernelILi128ELi128ELi4ELi2ELb1ELi5E": 31,      # faster than without: see the tile's comment
    r"gemm_mfma_kernelILi256ELi256ELi4ELi4ELb0ELi5E": 141,
}


def kernel_resources(code_object):
    """[(mangled name, vector registers, spilled vector registers)]"""
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code_object], check=True, capture_output=True, text=True).stdout
    found = []
    for kernel in notes.split("\n  - .a")[1:]:
        name, spilled, registers = (re.search(rf"\.{key}:\s+(\S+)", kernel) for key in (r"symbol", "vgpr_spill_count", "vgpr_count"))
        found.append((name.group(1), int(registers.group(1)), int(spilled.group(1))))
    assert len(found) > 100
    return found


def test_register_spills(code_object):
    over = {}
    for name, _, spilled in kernel_resources(code_object):
        if spilled > max((most for pattern, most in SPILLS.items() if re.search(pattern, name)), default=0):
            over[name] = spilled
    assert not over


# 256 threads without an LDS use that would limit them: a second wave on every SIMD is what hides the first one's loads.
TWO_WAVES = r"gemm_f32_kernel|rmsnorm_bwd_cols_kernel"


def test_registers_leave_two_waves(code_object):
    found = {name: registers for name, registers, _ in kernel_resources(code_object) if re.search(TWO_WAVES, name)}
    assert len(found) > 10
    assert not {name: registers for name, registers in found.items() if registers > 256}


REFUSALS = r"""
#include <cstdio>
#include "gemm_f32.h"
using namespace armt;
int main() {
  GemmShape s{};
  s.M = 72; s.N = 256; s.K = s.lda = s.ldb = 128; s.ldc = 256; s.n0 = 128; s.n1 = 64; s.ldr = 32; s.epi = EPI_QKV_ROPE;
  std::printf("%d", launch_gemm_f32(nullptr, 0, 0, s, nullptr) == hipSuccess);      // no groups: nothing to do, nothing to refuse
  return launch_gemm_f32(nullptr, 0, 1, s, nullptr) == hipErrorInvalidValue ? 0 : 1;
}
"""


def test_f32_rotation_needs_the_norm(tmp_path):
    """The plain fp32 product does not rotate: a shape that asks for it is refused on the host.  (Run without a GPU: nothing can be launched.)"""
    from paper_2506_05229_amd.build import CSRC
    (tmp_path / "refusals.hip").write_text(REFUSALS)
    flags = ["-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", f"-I{CSRC}"]
    subprocess.run(["/opt/rocm/bin/hipcc", *flags, "-o", tmp_path / "refusals", tmp_path / "refusals.hip"], check=True, capture_output=True)
    ran = subprocess.run([tmp_path / "refusals"], env={**os.environ, "HIP_VISIBLE_DEVICES": "-1"}, capture_output=True, text=True)
    assert ran.returncode == 0 and ran.stdout == "1"

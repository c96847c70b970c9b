"""Registers of the compiled kernels that launch rules count on (gfx950
listings; a SIMD has 512 vector registers per lane, so a wave that holds more
than 256 runs alone on it)."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_01565_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S", "-o", "-",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _registers(src):
    """{kernel: vector registers (VGPRs and AGPRs together)} of a source file."""
    r = subprocess.run([HIPCC, *FLAGS, os.path.join(CSRC, src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, name = {}, None
    for line in r.stdout.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = m.group(1)
        m = re.match(r"^; TotalNumVgprs: (\d+)", line)
        if m and name:
            out[name] = int(m.group(1))
    return out


@pytest.fixture(scope="module")
def registers():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    srcs = ["elementwise.hip", "gemm_bf16.hip"]
    with ThreadPoolExecutor(len(srcs)) as ex:
        return dict(zip(srcs, ex.map(_registers, srcs)))


def test_gemm_blocks_of_four_waves_run_two_per_cu(registers):
    regs = {k: v for k, v in registers["gemm_bf16.hip"].items() if "gemm_bf16_kernel" in k}
    four = {k: v for k, v in regs.items() if re.search(r"ILi128ELi(64ELi4ELi1|128ELi2ELi2)E", k)}
    assert len(regs) >= 10 and len(four) == 4  # 128x64 and 128x128, direct-to-LDS and register path
    assert max(four.values()) <= 256, four


def test_gemv_blocks_per_cu_are_the_compiled_ones(registers):
    """launch_gemv's round of resident blocks: the table in the source against the registers of every instance
    (blocks of four waves, so blocks per CU are waves per SIMD, eight at most)."""
    src = open(os.path.join(CSRC, "elementwise.hip")).read()
    maxc = [int(x) for x in re.search(r"kGemvMaxC\[\] = \{([\d, ]+)\}", src).group(1).split(",")]
    regs = registers["elementwise.hip"]
    for letter, name in (("t", "kGemvPerCuBf16"), ("f", "kGemvPerCuF32")):
        table = re.search(name + r"\[2\]\[7\] = \{\{([\d, ]+)\}, \{([\d, ]+)\}\}", src)
        for first in (0, 1):
            want = [int(x) for x in table.group(1 + first).split(",")]
            got = []
            for c in maxc:
                k = [v for n, v in regs.items() if f"gemv_kernelI{letter}Li{c}ELb{first}E" in n]
                assert len(k) == 1, (name, c, first)
                got.append(min(8, 512 // ((k[0] + 7) // 8 * 8)))
            assert got == want, (name, first, got)

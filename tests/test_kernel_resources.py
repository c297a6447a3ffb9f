"""Compile-only checks of the gfx950 code objects (no GPU needed): two mistakes that do not show up as
compile errors and that cost this code base dearly when they happened.

* A register array that the compiler cannot keep in registers (an array of HIP's uint4 struct behind a
  generic lambda, a dynamically indexed array) lands in scratch memory: the kernel still computes the
  right values, several times slower.  Every kernel must have a private segment of 0 bytes.
* Inline assembly next to MFMAs is not covered by the compiler's hazard handling (the wait states an MFMA
  needs after a VALU write of its operands): no kernel may contain an inline-assembly block.
"""
import glob
import os
import re
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = sorted(glob.glob(os.path.join(ROOT, "paper_2602_02711_amd", "csrc", "*.hip")))
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "--cuda-device-only", "-S"]
SCRATCH_ALLOWED = {}        # file name -> bytes per lane (none accepted at present)


def device_asm(src):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        proc = subprocess.run(["hipcc", *FLAGS, src, "-o", out], capture_output=True, text=True)
        assert proc.returncode == 0, proc.stderr[-2000:]
        return open(out).read()


@pytest.fixture(scope="module")
def listings():
    with ThreadPoolExecutor(max_workers=4) as pool:
        return dict(zip(SOURCES, pool.map(device_asm, SOURCES)))


def test_no_kernel_uses_scratch_memory(listings):
    for src, text in listings.items():
        sizes = [int(v) for v in re.findall(r"\.private_segment_fixed_size:\s*(\d+)", text)]
        limit = SCRATCH_ALLOWED.get(os.path.basename(src), 0)
        assert all(v <= limit for v in sizes), (os.path.basename(src), max(sizes))


def test_no_inline_assembly_in_kernels(listings):
    for src, text in listings.items():
        assert "#ASMSTART" not in text, os.path.basename(src)


def argument_bytes(text, kernel):
    """name -> end of the last byte that each instance of `kernel` loads from its arguments."""
    ends = {}
    for m in re.finditer(r"^(\S*%s\S*):\s*;" % kernel, text, re.M):
        body = text[m.end():text.index("s_endpgm", m.end())]
        words = {"": 1, "x2": 2, "x3": 3, "x4": 4, "x8": 8, "x16": 16}
        ends[m.group(1)] = max(int(off, 16) + 4 * words[n] for n, off in
                               re.findall(r"s_load_dword(x\d+)?\s+\S+, s\[0:1\], (0x[0-9a-f]+)", body))
    return ends


def test_one_row_kernel_reads_one_line_of_arguments(listings):
    # launches of a few microseconds: a second 64-byte line of arguments, fetched from memory, costs 0.2 .. 0.35 us of each
    text = next(t for src, t in listings.items() if os.path.basename(src) == "w3_gemv.hip")
    ends = argument_bytes(text, "w3_gemv_kernel")
    assert ends and all(v <= 64 for v in ends.values()), ends


def test_place_of_the_long_prefill_loop(tmp_path):
    # the main loop of the 256 x 256 INT4 group kernel without a residual, 2708 bytes: 1 .. 2 % slower where it begins 0, 4, 12 or 32 bytes
    # into a 64-byte line, 0.5 % at 48 and 56, than at 20, 28 or 40
    src = next(s for s in SOURCES if os.path.basename(s) == "gemm_w4_rescale.hip")
    obj, co = str(tmp_path / "k.o"), str(tmp_path / "k.co")
    llvm = "/opt/rocm/llvm/bin/"
    run = lambda *cmd: subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    run("hipcc", *[f for f in FLAGS if f != "-S"], "-c", src, "-o", obj)
    run(llvm + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + obj,
        "--output=" + co)
    text = run(llvm + "llvm-objdump", "-d", "--no-show-raw-insn", co)
    kernels = re.findall(r"<(\S*gemm_w4_rescale_kernelILi2ELi4ELi1ELi4ELi2ELi4ELb[01]ELb0ELb0E\S*)>:\n(.*?)\n\n", text, re.S)
    assert len(kernels) == 2                          # bf16 and fp32 output
    for name, body in kernels:
        back = [(int(a, 16) + 4 + (int(off) - 65536) * 4, int(a, 16)) for off, a in
                re.findall(r"s_cbranch_\S+ (\d+)\s*//\s*([0-9A-F]+):", body) if int(off) > 32767]
        first, end = back[0]
        assert 2000 < end - first < 4000 and first % 64 in (20, 28, 40), (name, first % 64, end - first)

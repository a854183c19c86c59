"""CPU-only: the kernels whose wavefronts wait for the K tiles of their private LDS rings by counting outstanding loads
count nothing but K tiles, whose loads are a fixed number of instructions."""
import os
import re
import subprocess

import pytest

from paper_2601_10639_amd import build

DECODE = r"gemm_decode_kernelINS_5ShapeILi(\d+)ELi(\d+)ELi\d+ELi(\d+)EEE"
F32 = r"gemm_f32_kernelILi(\d+)ELi\d+ELi(\d+)E"


@pytest.mark.parametrize("source,pattern", [("gemm_decode_bf16.hip", DECODE), ("kernels_f32.hip", F32)])
def test_waits_allow_for_no_loads_but_the_younger_k_tiles(source, pattern, tmp_path):
    out = str(tmp_path / "kernels.s")
    subprocess.run([build._hipcc(), *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out],
                   check=True, capture_output=True)
    seen = 0
    for name, body in re.findall(r"^(_Z\S+):[^\n]*\n(.*?)\.Lfunc_end", open(out).read(), re.S | re.M):
        m = re.search(pattern, name)
        if not m:
            continue
        if source.startswith("gemm_decode"):
            fa, fb, depth = map(int, m.groups())
            per_tile = 2 * (fa + fb)                      # 1 KB each: 16 rows of 128 bytes are two
        else:
            ts, depth = map(int, m.groups())
            per_tile = 2 * ts * 32 * 4 // 1024
        waits = [int(n) for block in re.findall(r";#ASMSTART(.*?);#ASMEND", body, re.S) for n in re.findall(r"vmcnt\((\d+)\)", block)]
        assert waits and max(waits) == (depth - 1) * per_tile, (name, waits)
        seen += 1
    assert seen >= 7


def test_waits_of_the_kernel_with_paired_k_halves(tmp_path):
    out = str(tmp_path / "kernels.s")
    subprocess.run([build._hipcc(), *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "gemm_decode_bf16.hip"),
                    "-o", out], check=True, capture_output=True)
    kernels = [(int(m.group(1)), m.group(2)) for m in
               re.finditer(r"^_Z\S+gemm_decode_kernelINS_9PairShapeILi\d+ELi(\d+)EEE[^\n]*:[^\n]*\n(.*?)\.Lfunc_end", open(out).read(), re.S | re.M)]
    assert kernels
    for depth, body in kernels:
        waits = [int(n) for block in re.findall(r";#ASMSTART(.*?);#ASMEND", body, re.S) for n in re.findall(r"vmcnt\((\d+)\)", block)]
        assert waits and max(waits) == (depth - 1) * 4, waits    # 16 rows of each operand: two loads each

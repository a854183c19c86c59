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


ONE_LAUNCH = r"ffn_decode_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)EE"


@pytest.fixture(scope="module")
def layer_kernels(tmp_path_factory):
    """((RG, KG, TQ, RD), lines) of each kernel of the layer in one launch, and their metadata (LDS, scratch, registers, spills)."""
    out = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    subprocess.run([build._hipcc(), *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "ffn_decode_bf16.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    bodies = {tuple(map(int, m.groups()[:4])): [line.strip() for line in m.group(5).split("\n")]
              for m in re.finditer(r"^_Z\S+" + ONE_LAUNCH + r"[^\n]*:[^\n]*\n(.*?)\.Lfunc_end", text, re.S | re.M)}
    meta = {tuple(map(int, m.groups()[1:5])): tuple(map(int, (m.group(1), *m.groups()[5:]))) for m in re.finditer(
        r"\.group_segment_fixed_size: (\d+)(?:(?!\.group_segment).)*?\.name: +_Z\S+" + ONE_LAUNCH +
        r"(?:(?!\.group_segment).)*?\.private_segment_fixed_size: (\d+).*?\.vgpr_count: +(\d+).*?\.vgpr_spill_count: (\d+)", text, re.S)}
    return bodies, meta


def test_two_workgroups_of_the_layer_in_one_launch_fit_a_compute_unit(layer_kernels):
    """Its workgroups wait for each other: two launches at a time have to be resident together (512 registers a SIMD lane, 160 KB of LDS)."""
    bodies, meta = layer_kernels
    assert set(meta) == set(bodies) == {(rg, kg, tq, 4 if kg <= 2 else 8) for rg in range(1, 5) for kg in range(1, 5) for tq in range(1, 5) if kg * tq <= 9}
    for kernel, (lds, scratch, registers, spills) in meta.items():
        assert 2 * lds <= 160 * 1024 and registers <= 512 // 4 and scratch == spills == 0, kernel   # 2 x 8 wavefronts on 4 SIMDs


def test_counted_waits_of_the_layer_in_one_launch(layer_kernels):
    """x is in LDS, and later H is stored, when no more loads are outstanding than are certainly younger: at least as many follow, with no
    branch between."""
    vmem = re.compile(r"(buffer|global)_(load|store|atomic)")
    for kernel, lines in layer_kernels[0].items():
        inside, waits = False, []
        for i, line in enumerate(lines):
            inside = "#ASMSTART" in line or inside and "#ASMEND" not in line
            m = re.match(r"s_waitcnt vmcnt\(([1-9]\d*)\)$", line)
            if inside and m:
                waits.append((i, int(m.group(1))))
        assert len(waits) == 2, (kernel, waits)
        for turn, (at, count) in enumerate(waits):
            if turn == 0:
                after = max(i for i, line in enumerate(lines[:at]) if re.match(r"buffer_load_dwordx4 .* lds$", line))
            else:
                after = max(i for i, line in enumerate(lines[:at]) if vmem.match(line) and "_store" in line)
                after = next(i for i in range(after, at) if re.match(r"\.LBB\S+:", lines[i]))     # behind the branches that store
            between = lines[after + 1:at]
            assert not any(re.match(r"\.LBB\S+:|s_c?branch", line) or "_store" in line for line in between), (kernel, turn)
            assert sum(bool(vmem.match(line)) for line in between) >= count, (kernel, turn, count)

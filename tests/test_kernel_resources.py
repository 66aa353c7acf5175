"""Register budget of the headline kernel, checked at compile time (no GPU): the tiled kernels are bound by vector-ALU
issue, and their 2 x 2 variants lose about a fifth of their throughput when they drop from four waves per SIMD to three.
Called routines count against a kernel's registers, so a change far from the hot loops can cost that wave; this test
recompiles the translation unit of the chained bench kernel with the compiler's resource remarks and checks them."""
import functools
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_10909_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_headline_kernel_keeps_four_waves_per_simd():
    cmd = ["hipcc", "-c", os.path.join(CSRC, "emulate_tiled_c1v1.hip"), "-o", os.devnull, "--offload-arch=gfx950", "-O3", "-fPIC",
           "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    # template arguments: 32 x 32 block, 2 x 2 per thread, 32 k staged, groups of 8, accumulator added exactly afterwards,
    # no fold, BF16 values: the kernel bench.py reports as "chained"
    name = "emulate_tiled_kernelILi32ELi32ELi2ELi2ELi32ELi8ELi1ELi0ELi1E"
    blocks = [b for b in out.stderr.split("Function Name:")[1:] if name in b.split("\n")[0]]
    assert len(blocks) == 1, "kernel not found in the resource remarks"
    get = lambda key: int(re.search(key + r":\s*(\d+)", blocks[0]).group(1))
    assert get(r"Occupancy \[waves/SIMD\]") >= 4, blocks[0]
    assert get("VGPRs Spill") == 0 and get("VGPRs") <= 128, blocks[0]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_scan_kernels_keep_their_products_in_registers():
    """The scan kernel's T-FDPA instantiations hold up to 64 products per thread: on BF16 operands, and on 16x16x16 and 32x32x8
    tiles of all operands, with or without twins, none of them may send registers to scratch memory (BF16 twins: once 121
    registers, launches of few sets took 1.3 times as long; FP16 on 16x16x16: 8, 2 to 4 %)."""
    cmd = ["hipcc", "-c", os.path.join(CSRC, "emulate_scan.hip"), "-o", os.devnull, "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-fPIC",
           "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    # template arguments: tile, k, BF16, T-FDPA, twins
    blocks = [b for b in out.stderr.split("Function Name:")[1:] if re.search(r"emulate_scan_kernelI(Li(16|32)ELi(8|16)ELb1E|Li16ELi16ELb0E|Li32ELi8ELb0E)Li0ELb[01]E", b.split("\n")[0])]
    assert len(blocks) == 10, "kernels not found in the resource remarks"
    for b in blocks:
        assert int(re.search(r"VGPRs Spill:\s*(\d+)", b).group(1)) == 0, b
    # TR-FDPA with its products kept, at four waves per SIMD: 15, 8 and no registers of a thread (three waves take longer from 2^14 tiles of 16x16x16 on)
    for tile, most in (("Li16ELi16E", 16), ("Li32ELi16E", 10), ("Li32ELi8E", 0)):
        blocks = [b for b in out.stderr.split("Function Name:")[1:] if "emulate_scan_kernelI" + tile + "Lb0ELi4E" in b.split("\n")[0]]
        assert len(blocks) == 1, "kernel not found in the resource remarks"
        assert int(re.search(r"VGPRs Spill:\s*(\d+)", blocks[0]).group(1)) <= most and int(re.search(r"Occupancy \[waves/SIMD\]:\s*(\d+)", blocks[0]).group(1)) >= 4, blocks[0]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_packed_kernels_need_no_scratch_memory():
    """The packed FP8 kernels run at four waves per SIMD with all their values in registers (with a routine of its own for groups far
    below their rows' products they once kept up to 36 registers, and that routine's results, in scratch memory)."""
    cmd = ["hipcc", "-c", os.path.join(CSRC, "emulate_packed.hip"), "-o", os.devnull, "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-fPIC",
           "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    blocks = [b for b in out.stderr.split("Function Name:")[1:] if "emulate_packed_kernel" in b.split("\n")[0]]
    # three pairs of types and, of equal types, two group lengths; two block sizes
    assert len(blocks) == 8, "kernels not found in the resource remarks"
    for b in blocks:
        get = lambda key: int(re.search(key + r":\s*(\d+)", b).group(1))
        assert get("VGPRs Spill") == 0 and get(r"ScratchSize \[bytes/lane\]") == 0 and get(r"Occupancy \[waves/SIMD\]") >= 4, b


@functools.lru_cache(maxsize=None)
def resource_remarks(source):
    cmd = ["hipcc", "-c", os.path.join(CSRC, source + ".hip"), "-o", os.devnull, "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-fPIC",
           "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    return out.stderr.split("Function Name:")[1:]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source,kernel,count,waves,spill", [
    ("emulate_packed_rd", "emulate_packed_rd_kernelILi\\dELi\\dELi2E", 6, 5, 0), ("emulate_packed_rd", "emulate_packed_rd_kernelILi\\dELi\\dELi4ELb0E", 3, 4, 0),
    ("emulate_packed_rd", "emulate_packed_rd_kernelILi\\dELi\\dELi4ELb1E", 3, 3, 0), ("emulate_small", "emulate_quad_kernel", 6, 4, 0),
    ("deviation", "deviation_tile_kernelILb[01]ELi1E", 4, 4, 0), ("deviation", "deviation_tile_kernelILb0ELi2E", 2, 4, 0),
    ("deviation", "deviation_tile_kernelILb1ELi2E", 2, 4, 4)])
def test_kernels_and_the_waves_they_are_measured_at(source, kernel, count, waves, spill):
    """Packed halves (two rows per lane, four, four with block scales), 4 x 4 tiles, and whole tiles of the deviation histogram: waves per
    SIMD, and registers in scratch memory, which only the 32-column kernel of FP8 operands has (2 of them)."""
    blocks = [b for b in resource_remarks(source) if re.search(kernel, b.split("\n")[0])]
    assert len(blocks) == count, "kernels not found in the resource remarks"
    for b in blocks:
        get = lambda key: int(re.search(key + r":\s*(\d+)", b).group(1))
        assert get("VGPRs Spill") <= spill and get(r"Occupancy \[waves/SIMD\]") >= waves, b

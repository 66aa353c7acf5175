"""Generators on the ranges where their kernels change route: whole Philox blocks or not, an unaligned output, block numbers that pass
2^32 inside a call; every family and the formats with a hardware conversion, against the CPU twin, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, gen as ogen
from gpu_utils import to_host
from test_gpu_parity import mm, NP  # noqa: F401  (fixture)

FORMATS = [fm.FP16, fm.BF16, fm.E4M3, fm.E5M2, fm.FP32]
# elements per tile, first tile, tiles, elements by which the output is moved off its alignment
RANGES = [(256, 3, 5, 0), (7, 3, 11, 0), (6, 5, 9, 1), (256, (1 << 26) - 1, 3, 0), (512, (1 << 25) - 1, 2, 0)]


@pytest.mark.parametrize("dtype", FORMATS)
def test_generator_ranges(mm, dtype):
    import torch
    torch_type = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[mm.ELEM_BYTES[dtype]]
    cases = [dict(family=f) for f in (mm.GEN_FINITE_BITS, mm.GEN_RANDOM_BITS, mm.GEN_SIGNED_ZEROS, mm.GEN_NORMAL)]
    cases += [dict(family=f, exp_lo=1, exp_hi=12, exp_zero=z) for f in (mm.GEN_UNIFORM_EXP, mm.GEN_CANCELLING) for z in (False, True)]
    cases += [dict(family=mm.GEN_NORMAL, scale_scope=mm.SCALE_FACTOR, scale_target=t) for t in (1e-3, 3e4)]       # subnormals, saturation
    for kw in cases:
        if dtype == fm.FP32 and kw["family"] == mm.GEN_CANCELLING:
            continue                                                  # (not defined there)
        for (ept, first, tiles, off) in RANGES:
            buf = torch.zeros(ept * tiles + 8, dtype=torch_type, device="cuda")
            mm.generate(buf[off:off + ept * tiles], dtype, ept, first, tiles, seed=77, operand=1, **kw)
            got = to_host(buf, NP[dtype])
            want = ogen.generate(ogen.GenParams(seed=77, operand=1, **kw), dtype, ept, first, tiles).reshape(-1)
            what = (dtype, kw, ept, first, tiles, off)
            assert np.array_equal(got[off:off + ept * tiles].astype(np.uint64), want.astype(np.uint64)), what
            assert not got[:off].any() and not got[off + ept * tiles:].any(), what


@pytest.mark.parametrize("dtype", FORMATS + [fm.E2M3])
def test_scaled_values(mm, dtype):
    # per-tile scaling on tiles of one wavefront, of a workgroup (one block per thread and several) and unaligned ones; per tensor
    import torch
    torch_type = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[mm.ELEM_BYTES[dtype]]
    for scope in (mm.SCALE_TILE, mm.SCALE_TENSOR):
        for (ept, first, tiles) in ((256, 3, 9), (252, 1, 5), (1024, 2, 3), (500, 1, 3), (4100, 1, 2), (7, 5, 11)):
            for family in (mm.GEN_NORMAL, mm.GEN_NORMAL_OUTLIERS, mm.GEN_UNIFORM):
                out = torch.zeros(ept * tiles, dtype=torch_type, device="cuda")
                kw = dict(family=family, scale_scope=scope, scale_target=100.0)
                mm.generate(out, dtype, ept, first, tiles, seed=78, operand=1, workspace=torch.zeros(1, dtype=torch.int64, device="cuda"), **kw)
                got = to_host(out, NP[dtype])
                want = ogen.generate(ogen.GenParams(seed=78, operand=1, **kw), dtype, ept, first, tiles).reshape(-1)
                assert np.array_equal(got.astype(np.uint64), want.astype(np.uint64)), (dtype, kw, ept, first, tiles)

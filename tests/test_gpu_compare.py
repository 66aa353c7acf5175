"""The comparison where few pairs differ or none: workgroups with nothing to fold beside one with a single pair."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, stats as ostats
from test_gpu_parity import dev_empty, mm, to_dev  # noqa: F401

# width: type, word, quiet NaN, another NaN, -0
WIDTHS = {16: (fm.FP16, np.uint16, 0x7E00, 0xFE01, 0x8000), 32: (fm.FP32, np.uint32, 0x7FC00000, 0xFFC00001, 0x80000000),
          64: (fm.FP64, np.uint64, 0x7FF8000000000000, 0xFFF8000000000001, 1 << 63)}


@pytest.mark.parametrize("width", sorted(WIDTHS))
@pytest.mark.parametrize("count,misalign", [(5, 0), (16384 * 3 + 7, 0), (16384 * 2 + 3, 1)])
def test_single_differing_pairs(mm, width, count, misalign):
    dtype, word, nan, nan2, minus_zero = WIDTHS[width]
    rng = np.random.default_rng(width + count)
    x = rng.integers(0, 1 << width, size=count + misalign, dtype=word)
    x[::97] = nan                                                    # equal NaNs: bucket 0, no mismatch
    st = dev_empty(mm.STATS_BYTES)
    mm.stats_reset(st)
    want = ostats.empty_stats()
    places = {0, 3, count // 2, count - 4, count - 1} | ({16383, 16384} if count > 16384 else set())
    base = 0
    for at in [None] + sorted(places):
        for a, b in ((1, 2), (0, minus_zero), (nan, nan2), (nan, 1)) if at is not None else ((0, 0),):
            x1, y1 = x.copy(), x.copy()
            if at is not None:
                x1[misalign + at], y1[misalign + at] = a, b
            mm.compare(to_dev(x1)[misalign:], to_dev(y1)[misalign:], count, st, index_base=base, d=dtype)
            want = ostats.compare(x1[misalign:], y1[misalign:], stats=want, index_base=base, width=width)
            assert mm.read_stats(st) == want, (at, hex(int(a)), hex(int(b)))
            base += count


@pytest.mark.parametrize("width", [16, 32])
@pytest.mark.parametrize("count", [4095, 4097, 16384, 64 * 4096 - 3, 64 * 4096 + 5, 65 * 16384 + 1])
def test_many_differing_pairs(mm, width, count):
    """Both sides of the workgroups' sizes, with patches that differ beside patches that do not (each wavefront's vectors equal, one pair
    of them different, all different): first index, largest distance (of numbers on either side of zero too) and every bucket."""
    dtype, word, nan, nan2, minus_zero = WIDTHS[width]
    rng = np.random.default_rng(width + count)
    x = rng.integers(0, 1 << width, size=count, dtype=word)
    y = x.copy()
    st = dev_empty(mm.STATS_BYTES)
    mm.stats_reset(st)
    want = ostats.empty_stats()
    for base, (lo, hi, frac) in enumerate(((count // 3, count, 0.0), (count - 1, count, 1.0), (count // 2, count, 0.01), (0, count, 1.0))):
        y = x.copy()
        pick = np.arange(lo, hi)[rng.random(hi - lo) < frac]
        y[pick] = rng.integers(0, 1 << width, size=len(pick), dtype=word)
        mm.compare(to_dev(x), to_dev(y), count, st, index_base=base * count, d=dtype)
        want = ostats.compare(x, y, stats=want, index_base=base * count, width=width)
        assert mm.read_stats(st) == want, (lo, hi, frac)


@pytest.mark.parametrize("count", [(1 << 23) - 2, 1 << 23, (1 << 23) + 1, (1 << 23) + (1 << 22) + 6])
def test_both_sides_of_the_loads_in_flight(mm, count):
    """Up to 2^23 pairs a thread has four loads per input in flight, beyond two: a differing patch at either end and in the middle, and
    pairs that differ in the vectors that are left over."""
    rng = np.random.default_rng(count & 0xFFFF)
    x = rng.integers(0, 1 << 32, size=count, dtype=np.uint32)
    y = x.copy()
    for lo, hi, frac in ((0, 3000, 0.5), (count // 2, count // 2 + 20000, 0.01), (count - 1100, count, 0.3)):
        pick = np.arange(lo, hi)[rng.random(hi - lo) < frac]
        y[pick] = rng.integers(0, 1 << 32, size=len(pick), dtype=np.uint32)
    st = dev_empty(mm.STATS_BYTES)
    mm.stats_reset(st)
    mm.compare(to_dev(x), to_dev(y), count, st, index_base=11)
    assert mm.read_stats(st) == ostats.compare(x, y, index_base=11)

"""GPU parity of the packed-binary16 kernel (T-FDPA on FP8 operands, F up to 17) against the CPU oracle, bit for bit: widths at both
ends of its range, both group lengths, block edges, the data that reach the ends of its window (rows whose large elements never
meet) and those that leave it (accumulators far above the products, NaN and infinities), which take its second route."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, o2lib
from oracle.fdpa import ModelParams, C_IN_GROUP
from oracle.rounding import RNE, RZ
from paper_2511_10909_amd import synth
from test_gpu_parity import gpu_emulate, assert_same, mm, make_case  # noqa: F401  (fixture)
from test_gpu_tiled import operands

PAIRS = [(fm.E4M3, fm.E5M2), (fm.E5M2, fm.E4M3), (fm.E4M3, fm.E4M3)]
# (the last: enough outputs for the 64 x 64 blocks)
SHAPES = [(17, 33, 32, 2), (40, 70, 64, 1), (64, 64, 96, 3), (95, 129, 64, 1), (1500, 1409, 64, 1)]


def spread_rows(rng, nb, m, n, k, ta, tb):
    """Rows whose elements lie within a few places of each other, most rows far from the format's top; some elements of A are
    raised where B's are lowered, so that the rows' largest elements do not meet."""
    A, B = synth.narrow_exponent_bits(rng, (nb, m, k), ta, 3, 6), synth.narrow_exponent_bits(rng, (nb, n, k), tb, 3, 6)
    ma, mb = {fm.E4M3: 3, fm.E5M2: 2}[ta], {fm.E4M3: 3, fm.E5M2: 2}[tb]
    top_a, top_b = {fm.E4M3: 14, fm.E5M2: 30}[ta], {fm.E4M3: 14, fm.E5M2: 30}[tb]
    A[:, ::2, 0::4] = (A[:, ::2, 0::4] & 0x80) | (top_a << ma)
    B[:, :, 0::4] &= 0x81
    B[:, ::2, 1::4] = (B[:, ::2, 1::4] & 0x80) | (top_b << mb)
    A[:, :, 1::4] &= 0x81
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 90, 150)
    return A, B, C


@pytest.mark.parametrize("ta,tb", PAIRS)
def test_packed_kernel(mm, ta, tb):
    rng = np.random.default_rng(9100 + 8 * ta + tb)
    for (m, n, k, nb) in SHAPES:
        for mode in ("narrow", "full", "special", "spread", "far"):
            if m > 1000 and mode in ("narrow", "far"):
                continue
            for L in ((16, 32) if ta == tb else (32,)):
                F = int(rng.choice([10, 13, 14, 16] + ([17] if L == 16 else [])))
                p = ModelParams(group_len=L, frac_bits=F, c_mode=C_IN_GROUP, out_round=int(rng.integers(0, 2)), ftz_in=bool(rng.integers(0, 3) == 0),
                                ftz_out=bool(rng.integers(0, 2)), nan_bits=0x7FFFFFFF)
                if p.out_round == RZ and F == 13:
                    p = p.with_(out_mant_bits=13)
                if mode == "spread":
                    A, B, C = spread_rows(rng, nb, m, n, k, ta, tb)
                else:
                    A, B, C = operands(rng, ta, tb, nb, m, n, k, mode if mode != "far" else "narrow")
                    if mode == "far":                      # accumulators from far below to far above the products
                        C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 60, 254)
                print("packed", ta, tb, (m, n, k, nb), mode, p, flush=True)
                want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
                got = gpu_emulate(mm, p, A, B, C, ta, tb, in_place=mode == "full")
                what = "packed %s %s %s" % ((m, n, k, nb), mode, p)
                assert "packed fp16 L=%d" % L in gpu_emulate.last_kernel, (what, gpu_emulate.last_kernel)
                assert gpu_emulate.last_kernel.startswith("tiled 64x64" if m > 1000 else "tiled 32x32"), gpu_emulate.last_kernel
                assert_same(got, want, what)


def test_packed_kernel_keeps_to_its_range(mm):
    # wider sums, other group lengths, narrow tiles, two E5M2 operands: the other kernels
    rng = np.random.default_rng(9200)
    for (m, n, k, L, F) in ((64, 64, 64, 32, 17), (64, 64, 64, 16, 14), (64, 64, 64, 8, 14), (64, 64, 64, 32, 9), (16, 16, 32, 32, 14), (64, 64, 48, 16, 14)):
        p = ModelParams(group_len=L, frac_bits=F, c_mode=C_IN_GROUP)
        A, B, C = operands(rng, fm.E4M3, fm.E5M2, 1, m, n, k, "special")
        want, _ = o2lib.emulate_mma(p, A, B, C, fm.E4M3, fm.E5M2)
        got = gpu_emulate(mm, p, A, B, C, fm.E4M3, fm.E5M2)
        assert "packed" not in gpu_emulate.last_kernel, gpu_emulate.last_kernel
        assert_same(got, want, "%s" % ((m, n, k, L, F),))


def one_large(rng, nb, m, n, k, ta, tb):
    """One element near the format's top per row and 32 k, the others (zeros and subnormals among them) as far below it as the format
    goes: groups of 16 without it, and groups whose two large elements do not meet, 14 places and more below the rows' products."""
    def rows(count, t):
        x = synth.narrow_exponent_bits(rng, (nb, count, k), t, 0, 1)
        place = rng.integers(0, 32, (nb, count, k // 32)) + 32 * np.arange(k // 32)
        np.put_along_axis(x, place, np.uint32({fm.E4M3: 0x76, fm.E5M2: 0x7B}[t]) | (rng.integers(0, 2, place.shape) << 7).astype(np.uint32), axis=2)
        return x
    return rows(m, ta), rows(n, tb), synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 90, 130)


@pytest.mark.parametrize("ta,tb", PAIRS)
def test_packed_kernel_where_large_elements_do_not_meet(mm, ta, tb):
    """With NaN and infinities in a few rows, columns and accumulators of the same wavefronts, and without."""
    rng = np.random.default_rng(9600 + 8 * ta + tb)
    for (rows, nb, m, n, k) in ((spread_rows, 4, 64, 48, 64), (one_large, 4, 64, 48, 64), (one_large, 1, 1500, 1412, 32)):
        for frac in (0.0, 0.0005, 0.05):
            for L in ((16, 32) if ta == tb else (32,)):
                A, B, C = rows(rng, nb, m, n, k, ta, tb)
                A = synth.sprinkle(rng, A, synth.SPECIAL_CODES[ta], frac)
                B = synth.sprinkle(rng, B, synth.SPECIAL_CODES[tb], frac)
                C = synth.sprinkle(rng, C, synth.SPECIAL_CODES[fm.FP32], frac)
                for F in (10, 16):
                    p = ModelParams(group_len=L, frac_bits=F, c_mode=C_IN_GROUP, out_round=RZ, out_mant_bits=13, ftz_in=frac == 0.0005, nan_bits=0x7FFFFFFF)
                    print("packed apart", rows.__name__, ta, tb, L, frac, p, flush=True)
                    want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
                    got = gpu_emulate(mm, p, A, B, C, ta, tb)
                    assert "packed fp16 L=%d" % L in gpu_emulate.last_kernel, gpu_emulate.last_kernel
                    assert_same(got, want, "packed apart %s %s %s" % (rows.__name__, frac, p))


# (m, n, k, tiles, side of the blocks): batches of at least 2^21 outputs, tiles below, at and above the sizes where 64 x 64 blocks pad too much
BATCHES = [(32, 32, 64, 2048, 32), (17, 33, 32, 3800, 32), (65, 40, 32, 808, 32), (64, 160, 32, 206, 32), (64, 224, 32, 147, 64), (33, 47, 32, 1408, 64),
           (48, 48, 32, 911, 64), (48, 48, 32, 910, 32)]


@pytest.mark.parametrize("m,n,k,nb,side", BATCHES)
def test_packed_kernel_on_batches_of_small_tiles(mm, m, n, k, nb, side):
    rng = np.random.default_rng(9300 + m)
    for (ta, tb), L in (((fm.E4M3, fm.E5M2), 32), ((fm.E4M3, fm.E4M3), 16)):
        p = ModelParams(group_len=L, frac_bits=14, c_mode=C_IN_GROUP)
        A, B, C = operands(rng, ta, tb, nb, m, n, k, "special")
        print("packed batch", ta, tb, (m, n, k, nb), p, flush=True)
        want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
        got = gpu_emulate(mm, p, A, B, C, ta, tb)
        assert_same(got, want, "packed batch %s %s" % ((m, n, k, nb), p))
        assert gpu_emulate.last_kernel == "tiled %dx%d packed fp16 L=%d" % (side, side, L), gpu_emulate.last_kernel

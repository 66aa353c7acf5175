"""GPU parity of the packed-binary16 kernel (T-FDPA on FP8 operands, F up to 17) against the CPU oracle, bit for bit: widths at both
ends of its range, both group lengths, block edges, the data that reach the ends of its window (rows whose large elements never
meet) and those that leave it (accumulators far above the products, NaN and infinities), which take its second route."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, o2lib
from oracle.fdpa import ModelParams, C_IN_GROUP, C_AFTER_EXACT, C_AFTER_RD
from oracle.rounding import RNE, RZ
from gpu_utils import to_dev, to_host
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


# pair, m, n, k, L, F, switches: wider and narrower sums, other group lengths, k off the staged 32, narrow tiles, two E5M2 operands, other families
OUT_OF_RANGE = [((fm.E4M3, fm.E5M2), 64, 64, 64, 32, 17, {}), ((fm.E4M3, fm.E5M2), 64, 64, 64, 32, 9, {}), ((fm.E4M3, fm.E4M3), 64, 64, 64, 16, 18, {}),
                ((fm.E4M3, fm.E5M2), 64, 64, 64, 16, 14, {}), ((fm.E5M2, fm.E4M3), 64, 64, 64, 16, 14, {}), ((fm.E4M3, fm.E5M2), 64, 64, 64, 8, 14, {}),
                ((fm.E4M3, fm.E4M3), 64, 64, 48, 16, 14, {}), ((fm.E4M3, fm.E5M2), 16, 64, 32, 32, 14, {}), ((fm.E4M3, fm.E5M2), 64, 16, 32, 32, 14, {}),
                ((fm.E5M2, fm.E5M2), 64, 64, 64, 32, 14, {}), ((fm.E5M2, fm.E5M2), 64, 64, 64, 16, 14, {}),
                ((fm.E4M3, fm.E5M2), 64, 64, 64, 32, 14, dict(c_mode=C_AFTER_EXACT)),
                ((fm.E4M3, fm.E5M2), 64, 64, 64, 32, 14, dict(c_mode=C_AFTER_RD, frac_bits2=31, skip_zero_terms=True, zero_result_positive=True)),
                ((fm.FP16, fm.E4M3), 64, 64, 64, 32, 14, {})]


@pytest.mark.parametrize("case", range(len(OUT_OF_RANGE)))
def test_packed_kernel_keeps_to_its_range(mm, case):
    (ta, tb), m, n, k, L, F, switches = OUT_OF_RANGE[case]
    rng = np.random.default_rng(9200 + case)
    p = ModelParams(**dict(dict(group_len=L, frac_bits=F, c_mode=C_IN_GROUP), **switches))
    A, B, C = operands(rng, ta, tb, 1, m, n, k, "special")
    print("not packed", OUT_OF_RANGE[case], flush=True)
    want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
    got = gpu_emulate(mm, p, A, B, C, ta, tb)
    assert "packed" not in gpu_emulate.last_kernel, gpu_emulate.last_kernel
    assert_same(got, want, "%s" % (OUT_OF_RANGE[case],))


def test_fp16_outputs_keep_to_the_other_kernels(mm):
    rng = np.random.default_rng(9250)
    p = ModelParams(group_len=32, frac_bits=14, c_mode=C_IN_GROUP, nan_bits=0x7FFF)
    A, B, _ = operands(rng, fm.E4M3, fm.E5M2, 1, 64, 64, 64, "special")
    C = synth.random_bits(rng, (1, 64, 64), fm.FP16)
    want, _ = o2lib.emulate_mma(p, A, B, C, fm.E4M3, fm.E5M2, tc=fm.FP16)
    got = gpu_emulate(mm, p, A, B, C, fm.E4M3, fm.E5M2, tc=fm.FP16)
    assert "packed" not in gpu_emulate.last_kernel, gpu_emulate.last_kernel
    assert_same(got, want, "FP16 outputs")


def emulate_at(mm, p, A, B, C, ta, tb, offset, in_place):
    """The emulation with C and D `offset` words off a 16-byte boundary and sixteen guard words on either side of D."""
    import torch
    (nb, m, k), n = A.shape, B.shape[1]
    h = mm.model_create(group_len=p.group_len, frac_bits=p.frac_bits, c_mode=p.c_mode, out_round=p.out_round, ftz_in=p.ftz_in, ftz_out=p.ftz_out,
                        nan_bits=p.nan_bits, out_mant_bits=p.out_mant_bits)
    try:
        dA, dB = to_dev(A.astype(np.uint8)), to_dev(B.astype(np.uint8))
        count = nb * m * n
        bufs = [torch.full((count + 36,), -559038737, dtype=torch.int32, device="cuda") for _ in range(1 if in_place else 2)]
        views = [b[16 + offset:16 + offset + count] for b in bufs]
        views[0].copy_(to_dev(C.astype(np.uint32)).reshape(-1))
        mm.emulate_mma(h, dA, dB, views[0], views[-1], m, n, k, nb, (ta, tb, fm.FP32, fm.FP32))
        kernel = mm.last_kernel()
        out = to_host(bufs[-1], np.uint32)
        assert (out[:16 + offset] == 0xDEADBEEF).all() and (out[16 + offset + count:] == 0xDEADBEEF).all(), "written outside D"
        return out[16 + offset:16 + offset + count].reshape(nb, m, n), kernel
    finally:
        mm.model_destroy(h)


# n a multiple of four (C and D move in 128-bit words) with the right edge inside a block, both block sizes, one and several tiles
WIDE = [(40, 36, 64, 2, 32), (17, 100, 32, 1, 32), (64, 64, 32, 3, 32), (1500, 1412, 64, 1, 64), (1090, 1000, 32, 2, 64)]


@pytest.mark.parametrize("m,n,k,nb,side", WIDE)
@pytest.mark.parametrize("ta,tb", PAIRS)
def test_packed_kernel_with_wide_stores(mm, m, n, k, nb, side, ta, tb):
    rng = np.random.default_rng(9500 + m + 8 * ta + tb)
    for mode in ("full", "special", "spread"):
        L = int(rng.choice([16, 32])) if ta == tb else 32
        p = ModelParams(group_len=L, frac_bits=14, c_mode=C_IN_GROUP, out_round=int(rng.integers(0, 2)), ftz_out=bool(rng.integers(0, 2)), nan_bits=0x7FFFFFFF)
        A, B, C = spread_rows(rng, nb, m, n, k, ta, tb) if mode == "spread" else operands(rng, ta, tb, nb, m, n, k, mode)
        want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
        for offset in ((0, 1) if m < 1000 else (0,)):
            print("packed wide", ta, tb, (m, n, k, nb), mode, offset, p, flush=True)
            got, kernel = emulate_at(mm, p, A, B, C, ta, tb, offset, mode == "full")
            assert_same(got, want, "packed wide %s %s %d %s" % ((m, n, k, nb), mode, offset, p))
            assert kernel == "tiled %dx%d packed fp16 L=%d" % (side, side, L), kernel


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


@pytest.mark.parametrize("ta,tb", PAIRS)
@pytest.mark.parametrize("ftz_in", [False, True])
def test_packed_kernel_sums_of_zeros_are_positive(mm, ta, tb, ftz_in):
    """Products that are zeros of either sign and negative accumulators that the alignment cuts to zero (or are -0): the sum is +0."""
    rng = np.random.default_rng(9700 + 8 * ta + tb)
    for L in ((16, 32) if ta == tb else (32,)):
        A = (rng.integers(0, 2, (2, 40, 64)) << 7).astype(np.uint32)                       # zeros of both signs
        B = synth.narrow_exponent_bits(rng, (2, 36, 64), tb, 1, 12)
        A[1, ::2] |= 0x80                                                                # rows of negative zeros alone
        B[1, ::2] &= 0x7F
        C = np.choose(rng.integers(0, 4, (2, 40, 36)), [0x80000000, 0x80000001, 0x8D000000, 0x80800000]).astype(np.uint32)
        p = ModelParams(group_len=L, frac_bits=14, c_mode=C_IN_GROUP, out_round=int(L == 16), ftz_in=ftz_in)
        print("packed zeros", ta, tb, p, flush=True)
        want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
        got = gpu_emulate(mm, p, A, B, C, ta, tb)
        assert "packed fp16 L=%d" % L in gpu_emulate.last_kernel, gpu_emulate.last_kernel
        assert not want.any()
        assert_same(got, want, "packed zeros %s" % p)


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

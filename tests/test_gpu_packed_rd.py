"""GPU parity of the packed-binary16 kernel for GTR-FDPA in halves of eight (FP8 operands, F of 10 to 17) against the CPU oracle, bit for
bit: widths at both ends, maxima inside and below the window that one factor scales, zeros in and out of the maxima, special values,
block scales, both splits of a block over wavefronts, and what stays with the other kernels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, o2lib
from oracle.fdpa import ModelParams, C_AFTER_RD, SPLIT_HALVES
from paper_2511_10909_amd import synth
from test_gpu_parity import mm, gpu_emulate, assert_same  # noqa: F401
from test_gpu_scaled import gpu_emulate_scaled

BASE = ModelParams(group_len=16, frac_bits=13, frac_bits2=31, c_mode=C_AFTER_RD, split=SPLIT_HALVES, frac_bits_merge=24, frac_bits_acc=24,
                   skip_zero_terms=True, f2_at_leading_bit=True, zero_result_positive=True, acc_special_truncation=True, sum_drop_distance=28,
                   nan_bits=0xFFC00000, wide_products=True)
MODELS = [BASE, BASE.with_(frac_bits=10, frac_bits_merge=25, sum_drop_distance=27), BASE.with_(frac_bits=17, frac_bits_acc=20), BASE.with_(frac_bits=12, frac_bits_merge=12, skip_zero_terms=False),
          BASE.with_(frac_bits=14, acc_special_truncation=False, zero_result_positive=False, frac_bits2=24), BASE.with_(frac_bits=17, frac_bits_merge=17, sum_drop_distance=3)]
PAIRS = [(fm.E4M3, fm.E4M3), (fm.E4M3, fm.E5M2), (fm.E5M2, fm.E4M3)]
LARGE = {fm.E4M3: 0x7E, fm.E5M2: 0x7B}


def operands(rng, ta, tb, nb, m, n, k, mode):
    mid = {fm.E4M3: (3, 11), fm.E5M2: (11, 19)}
    if mode == "mid":
        A, B = synth.narrow_exponent_bits(rng, (nb, m, k), ta, *mid[ta]), synth.narrow_exponent_bits(rng, (nb, n, k), tb, *mid[tb])
    else:
        A, B = synth.random_bits(rng, (nb, m, k), ta), synth.random_bits(rng, (nb, n, k), tb)
        if mode != "bits":
            finite = lambda X, t: np.where((X & 0x7F) > LARGE[t], LARGE[t], X).astype(X.dtype)
            A, B = finite(A, ta), finite(B, tb)
        if mode == "apart":              # large elements that never meet, tiny and zero ones elsewhere: maxima far below the largest elements'
            A, B = A & 0x87, B & 0x87
            A[..., 0::4], B[..., 1::4] = LARGE[ta], LARGE[tb]
            B[..., 0::4] = np.where(rng.random(B[..., 0::4].shape) < 0.7, 0, 1)
            A[..., 1::4] = np.where(rng.random(A[..., 1::4].shape) < 0.7, 0x80, 1)
        if mode == "zeros":
            A[rng.random(A.shape) < 0.7] = 0
            B[rng.random(B.shape) < 0.5] = 0x80
            A[0, 0], B[-1, -1] = 0, 0
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 100, 150)
    if mode == "bits":
        C = synth.sprinkle(rng, C, synth.SPECIAL_CODES[fm.FP32], 0.05)
    if mode == "zeros":
        C[rng.random(C.shape) < 0.3] = 0x80000000
        C[rng.random(C.shape) < 0.1] = 0x00000007
    return A, B, C


@pytest.mark.parametrize("ta,tb", PAIRS)
@pytest.mark.parametrize("mode", ["mid", "finite", "bits", "apart", "zeros"])
def test_packed_halves(mm, ta, tb, mode):
    rng = np.random.default_rng(7000 + 10 * ta + tb)
    for nb, m, n, k, rows in ((3, 16, 16, 32, 2), (2, 48, 80, 96, 2), (4100, 16, 16, 32, 4), (17, 256, 256, 64, 4)):
        A, B, C = operands(rng, ta, tb, nb, m, n, k, mode)
        for p in MODELS if rows == 2 else MODELS[:2]:
            print("packed halves", ta, tb, (nb, m, n, k), mode, p, flush=True)
            want, _ = o2lib.emulate_mma(p, A, B, C, ta, tb)
            got = gpu_emulate(mm, p, A, B, C, ta, tb)
            assert "packed halves r%d" % rows in gpu_emulate.last_kernel, gpu_emulate.last_kernel
            assert_same(got, want, "%s %s %s" % ((nb, m, n, k), mode, p))


# tiles, m, n, k, rows per lane: either side of 768 blocks, workgroups of four wavefronts that are not full, blocks of tiles that are not
# square (819 of them; 1152 and 640, which are dealt to the XCDs in turn)
GRIDS = [(767, 16, 16, 32, 2), (768, 16, 16, 32, 4), (769, 16, 16, 32, 4), (770, 16, 16, 32, 4), (13, 112, 144, 64, 4), (24, 96, 128, 32, 4), (20, 32, 256, 32, 2)]


@pytest.mark.parametrize("nb,m,n,k,rows", GRIDS)
@pytest.mark.parametrize("scaled", [False, True])
def test_packed_halves_grids(mm, nb, m, n, k, rows, scaled):
    rng = np.random.default_rng(7300 + nb + m + n)
    ta, tb = fm.E4M3, fm.E5M2
    A, B, C = operands(rng, ta, tb, nb, m, n, k, "bits")
    print("packed halves", (nb, m, n, k), "scaled" if scaled else "", flush=True)
    if scaled:
        SA, SB = (rng.integers(100, 150, size=(nb, x, k // 32)).astype(np.uint8) for x in (m, n))
        want, got = o2lib.emulate_mma_scaled(BASE, A, B, C, SA, SB, 32, ta, tb)[0], gpu_emulate_scaled(mm, BASE, A, B, C, SA, SB, 32, ta, tb)
    else:
        want, got = o2lib.emulate_mma(BASE, A, B, C, ta, tb)[0], gpu_emulate(mm, BASE, A, B, C, ta, tb)
    assert "packed halves r%d" % rows in mm.last_kernel(), mm.last_kernel()
    assert_same(got, want, "%s" % ((nb, m, n, k),))


@pytest.mark.parametrize("ta,tb", PAIRS)
@pytest.mark.parametrize("mode", ["mid", "bits", "zeros"])
def test_packed_halves_with_block_scales(mm, ta, tb, mode):
    rng = np.random.default_rng(7100 + 10 * ta + tb)
    for nb, m, n, k in ((3, 16, 16, 128), (2, 32, 48, 64), (4100, 16, 16, 32)):
        A, B, C = operands(rng, ta, tb, nb, m, n, k, mode)
        SA, SB = rng.integers(100, 150, size=(nb, m, k // 32)).astype(np.uint8), rng.integers(0, 255, size=(nb, n, k // 32)).astype(np.uint8)
        SA[0, 0, 0], SB[-1, -1, -1] = 255, 255
        for p in MODELS[:3] if nb < 100 else MODELS[:1]:
            print("packed halves scaled", ta, tb, (nb, m, n, k), mode, p, flush=True)
            want, _ = o2lib.emulate_mma_scaled(p, A, B, C, SA, SB, 32, ta, tb)
            got = gpu_emulate_scaled(mm, p, A, B, C, SA, SB, 32, ta, tb)
            assert "packed halves" in mm.last_kernel(), mm.last_kernel()
            assert_same(got, want, "%s %s %s" % ((nb, m, n, k), mode, p))


# pair, m, n, k, switches, scaled: widths, lengths, splits and shapes of other kernels
OTHERS = [((fm.E5M2, fm.E5M2), 16, 16, 32, {}, 0), ((fm.E4M3, fm.E4M3), 16, 16, 48, {}, 0), ((fm.E4M3, fm.E4M3), 20, 16, 32, {}, 0),
          ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(frac_bits=9), 0), ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(frac_bits=18), 0),
          ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(frac_bits=14, frac_bits_merge=13), 0), ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(group_len=8), 0),
          ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(sum_drop_distance=0), 0), ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(ftz_in=True), 0),
          ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(out_round=1), 0), ((fm.E4M3, fm.E5M2), 16, 16, 32, dict(ftz_out=True), 0),
          ((fm.E4M3, fm.E4M3), 16, 16, 64, dict(wide_products=False), 32), ((fm.E4M3, fm.E4M3), 16, 16, 64, {}, 16), ((fm.E4M3, fm.E4M3), 16, 16, 128, {}, 64)]


@pytest.mark.parametrize("case", range(len(OTHERS)))
def test_packed_halves_keep_to_their_range(mm, case):
    (ta, tb), m, n, k, switches, block = OTHERS[case]
    rng = np.random.default_rng(7200 + case)
    p = BASE.with_(**switches)
    A, B, C = operands(rng, ta, tb, 2, m, n, k, "bits")
    print("not packed halves", OTHERS[case], flush=True)
    if block:
        SA, SB = (rng.integers(100, 150, size=(2, x, k // block)).astype(np.uint8) for x in (m, n))
        want, got = o2lib.emulate_mma_scaled(p, A, B, C, SA, SB, block, ta, tb)[0], gpu_emulate_scaled(mm, p, A, B, C, SA, SB, block, ta, tb)
    else:
        want, got = o2lib.emulate_mma(p, A, B, C, ta, tb)[0], gpu_emulate(mm, p, A, B, C, ta, tb)
    assert "packed" not in mm.last_kernel(), mm.last_kernel()
    assert_same(got, want, "%s" % (OTHERS[case],))

"""Sec. 6.2.4 on the GPU: the truncating variant of TR-FDPA (rd_toward_zero) in the general and in the tiled kernels
against the rational oracle, mmaemu_deviation_sample against oracle/exact.py (integers bit-exact, the three binary64
sums to 1e-9), the constant-factor generator against its CPU twin, and the experiment itself as a device workload."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import formats as fm, o2lib, gen as ogen
from oracle.exact import deviation_hist
from oracle.fdpa import ModelParams, C_AFTER_RD, C_AFTER_RD_EVEN_ODD, SPLIT_HALVES, SPLIT_QUARTERS, SPLIT_EVEN_ODD
from paper_2511_10909_amd import synth
from gpu_utils import to_dev, to_host
from o1_jobs import run_pool
from test_gpu_parity import mm, gpu_emulate, assert_same  # noqa: F401

TRZ = ModelParams(group_len=8, frac_bits=24, frac_bits2=31, c_mode=C_AFTER_RD, rd_toward_zero=True)


def close(a, b):
    return abs(a - b) <= 1e-9 * max(abs(a), abs(b), 1e-300)


def same_hist(got, want, what):
    for key in ("n_samples", "n_skipped", "n_negative", "n_zero", "n_positive", "bins"):
        assert got[key] == want[key], (what, key, got[key], want[key])
    for key in ("sum", "sum_abs", "sum_sq"):
        assert close(got[key], want[key]), (what, key, got[key], want[key])


def test_truncating_variant_matches_the_rational_oracle(mm):
    rng = np.random.default_rng(777)
    cases = [("unsplit fp16, ragged (general)", TRZ, fm.FP16, (5, 12, 20, 16), "general"),
             ("unsplit bf16, ragged (general)", TRZ.with_(frac_bits=20, frac_bits2=27, out_round=1), fm.BF16, (5, 12, 20, 16), "general"),
             ("even/odd fp8 (general)", TRZ.with_(c_mode=C_AFTER_RD_EVEN_ODD, group_len=16), fm.E5M2, (5, 12, 20, 32), "general"),
             ("halves, F_m = 20 (general)", TRZ.with_(split=SPLIT_HALVES, frac_bits_merge=20, group_len=8), fm.FP16, (4, 16, 16, 16), "general"),
             ("quarters (general)", TRZ.with_(split=SPLIT_QUARTERS, frac_bits=13, group_len=16), fm.E4M3, (4, 16, 16, 32), "general"),
             ("leading-bit F2 rule, zero terms skipped (general)", TRZ.with_(f2_at_leading_bit=True, skip_zero_terms=True, zero_result_positive=True), fm.BF16, (4, 16, 16, 16), "general"),
             ("special truncation, drop distance (tiled)", TRZ.with_(acc_special_truncation=True, sum_drop_distance=28), fm.FP16, (2, 32, 32, 16), "tiled"),
             ("unsplit fp16 32x32x8 (tiled)", TRZ, fm.FP16, (2, 32, 32, 8), "tiled"),
             ("unsplit bf16 16x16x16 (tiled)", TRZ, fm.BF16, (6, 16, 16, 16), "tiled"),
             ("unsplit fp8 16x16x32 (tiled)", TRZ.with_(group_len=16, frac_bits=13, frac_bits2=24), fm.E4M3, (6, 16, 16, 32), "tiled")]
    gpu, jobs = [], []
    for idx, (name, p, t, (nb, m, n, k), route) in enumerate(cases):
        A = synth.narrow_exponent_bits(rng, (nb, m, k), t, *((8, 22) if t != fm.BF16 and t != fm.E4M3 else ((120, 134) if t == fm.BF16 else (3, 12))))
        B = synth.narrow_exponent_bits(rng, (nb, n, k), t, *((8, 22) if t != fm.BF16 and t != fm.E4M3 else ((120, 134) if t == fm.BF16 else (3, 12))))
        C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 110, 140)
        if idx % 2:
            A = synth.sprinkle(rng, A, synth.SPECIAL_CODES[t], 0.01)
            C = synth.sprinkle(rng, C, synth.SPECIAL_CODES[fm.FP32], 0.01)
        got = gpu_emulate(mm, p, A, B, C, t, t)
        assert gpu_emulate.last_kernel.startswith(route), (name, gpu_emulate.last_kernel)
        gpu.append(got)
        jobs.append((dataclasses.asdict(p), A, B, C, t, t, None, None, 0))
        # the switch matters on these inputs: the printed algorithm differs somewhere
        rd = gpu_emulate(mm, p.with_(rd_toward_zero=False), A, B, C, t, t)
        assert (rd != got).any(), name
    want = run_pool(jobs, workers=12)
    for (name, *_), g, w in zip(cases, gpu, want):
        assert g.size >= 1000
        bad = np.argwhere(g != w)
        assert len(bad) == 0, "%s: %d of %d differ, first at %s: gpu %08x oracle %08x" % (name, len(bad), g.size, tuple(bad[0]), g[tuple(bad[0])], w[tuple(bad[0])])


def test_truncating_variant_block_scaled(mm):
    from test_gpu_scaled import gpu_emulate_scaled
    from oracle.fdpa import emulate_mma as o1
    rng = np.random.default_rng(778)
    p = TRZ.with_(group_len=16, frac_bits=13, frac_bits2=31, split=SPLIT_HALVES, frac_bits_merge=24, wide_products=True)
    nb, m, n, k, block = 2, 12, 11, 32, 32
    A, B = synth.random_bits(rng, (nb, m, k), fm.E4M3), synth.random_bits(rng, (nb, n, k), fm.E5M2)
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 100, 150)
    SA = rng.integers(110, 140, size=(nb, m, k // block)).astype(np.uint8)
    SB = rng.integers(110, 140, size=(nb, n, k // block)).astype(np.uint8)
    got = gpu_emulate_scaled(mm, p, A, B, C, SA, SB, block, fm.E4M3, fm.E5M2)
    want = o1(p, A, B, C, fm.E4M3, fm.E5M2, SA=SA, SB=SB, block=block)
    assert np.array_equal(got, want)


def test_constant_factor_generator_matches_cpu_twin(mm):
    import torch
    for dtype, np_t, ept, nt in ((fm.FP16, np.uint16, 256, 37), (fm.BF16, np.uint16, 100, 9), (fm.FP32, np.uint32, 1024, 5)):
        out = torch.empty(nt * ept, dtype={np.uint16: torch.int16, np.uint32: torch.int32}[np_t], device="cuda")
        mm.generate(out, dtype, ept, 3, nt, mm.GEN_NORMAL, seed=9, operand=1, scale_scope=mm.SCALE_FACTOR, scale_target=1000.0)
        want = ogen.generate(ogen.GenParams(family=ogen.GEN_NORMAL, seed=9, operand=1, scale_scope=ogen.SCALE_FACTOR, scale_target=1000.0),
                             dtype, ept, 3, nt).ravel()
        assert np.array_equal(to_host(out, np_t).astype(np.uint32), want.astype(np.uint32))


def dev_hist(mm, A, B, C, D, ta, tb, stride, bin_exp, calls=1):
    import torch
    h = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
    mm.deviation_hist_reset(h)
    nb, m, k = A.shape
    n = B.shape[1]
    dA, dB, dD = to_dev(A), to_dev(B), to_dev(D)
    dC = to_dev(C) if C is not None else None
    for _ in range(calls):
        mm.deviation_sample(dA, dB, dC, dD, m, n, k, nb, (ta, tb, fm.FP32, fm.FP32), stride, bin_exp, h)
    return mm.read_deviation_hist(h)


def test_deviation_sample_matches_oracle(mm):
    rng = np.random.default_rng(4)
    for idx, (ta, tb, shape, stride, bin_exp, with_c) in enumerate((
            (fm.FP16, fm.FP16, (5, 32, 32, 8), 1, -5, True), (fm.BF16, fm.BF16, (7, 16, 16, 16), 7, -12, False),
            (fm.E4M3, fm.E5M2, (3, 16, 16, 32), 3, -9, True), (fm.FP16, fm.BF16, (2, 9, 13, 5), 1, 2, True),
            (fm.E2M3, fm.E2M1, (4, 16, 16, 64), 5, -6, True), (fm.BF16, fm.BF16, (3, 16, 16, 8), 1, 0, True))):
        nb, m, n, k = shape
        lo_hi = {fm.FP16: (10, 24), fm.BF16: (118, 132), fm.E4M3: (3, 12), fm.E5M2: (10, 20), fm.E2M3: (0, 3), fm.E2M1: (0, 3)}
        A = synth.narrow_exponent_bits(rng, (nb, m, k), ta, *lo_hi[ta])
        B = synth.narrow_exponent_bits(rng, (nb, n, k), tb, *lo_hi[tb])
        C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 118, 132) if with_c else None
        if idx == 5:         # whole exponent range: many sums leave the pair of binary64 numbers for the wide accumulator
            A = synth.random_bits(rng, (nb, m, k), ta)
            B = synth.random_bits(rng, (nb, n, k), tb)
            C = synth.random_bits(rng, (nb, m, n), fm.FP32)
        if idx == 0:
            A = synth.sprinkle(rng, A, synth.SPECIAL_CODES[ta], 0.003)
            C = synth.sprinkle(rng, C, synth.SPECIAL_CODES[fm.FP32], 0.01)
        p = ModelParams(group_len=k, frac_bits=[24, 10, 13, 6, 30, 24][idx], frac_bits2=31, c_mode=C_AFTER_RD)
        D = o2lib.emulate_mma(p, A, B, C if with_c else np.zeros((nb, m, n), np.uint32), ta, tb)[0]
        if idx == 1:
            D[0, 0, :4] = [0x7F800000, 0x7FC00000, 0x00000001, 0x80000001]        # skipped; tiny outputs, far off
        got = dev_hist(mm, A, B, C, D, ta, tb, stride, bin_exp, calls=2 if idx == 2 else 1)
        want = deviation_hist(A, B, C, D, ta, tb, stride, bin_exp)
        if idx == 2:
            want = deviation_hist(A, B, C, D, ta, tb, stride, bin_exp, hist=want)
        same_hist(got, want, (ta, tb, shape))
        assert got["n_samples"] + got["n_skipped"] == (2 if idx == 2 else 1) * ((nb * m * n + stride - 1) // stride)
        if idx == 0:
            assert got["n_skipped"] > 0 and len([b for b in got["bins"] if b]) > 8


@pytest.mark.parametrize("ta,tb,shape,stride,c_offset", [
    (fm.FP16, fm.FP16, (3, 5, 4, 8), 1, 0), (fm.FP16, fm.E5M2, (1, 3, 4, 8192), 1, 0), (fm.FP16, fm.FP16, (1, 2, 4, 8200), 1, 0),
    (fm.E5M2, fm.E5M2, (2, 3, 8, 17), 1, 0), (fm.FP16, fm.FP16, (4, 7, 6, 8), 1, 0), (fm.FP16, fm.FP16, (3, 5, 8, 12), 1, 1),
    (fm.E4M3, fm.E4M3, (3, 4, 8, 16), 3, 0)])
def test_deviation_sample_split_sum(mm, ta, tb, shape, stride, c_offset):
    """Products at both ends of the narrow types' ranges (the split sum's two halves full), the k at which the split ends,
    rows of whole fours and rows that are not, an accumulator that is not 16-byte aligned (one output per thread: few outputs)."""
    import torch
    rng = np.random.default_rng(5 + shape[3])
    nb, m, n, k = shape
    A, B = synth.random_bits(rng, (nb, m, k), ta), synth.random_bits(rng, (nb, n, k), tb)
    big = {fm.FP16: 0x7BFF, fm.E5M2: 0x7B, fm.E4M3: 0x7E}
    A = np.where(rng.random(A.shape) < 0.4, np.where(rng.random(A.shape) < 0.5, big[ta], 1), A).astype(A.dtype)
    B = np.where(rng.random(B.shape) < 0.4, np.where(rng.random(B.shape) < 0.5, big[tb], 1), B).astype(B.dtype)
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 90, 160)
    D = o2lib.emulate_mma(ModelParams(group_len=k, frac_bits=24), A, B, C, ta, tb)[0]
    D[0, 0, 0] = 0x7F800000
    h = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
    mm.deviation_hist_reset(h)
    dC = to_dev(np.concatenate([np.zeros(c_offset, np.uint32), C.ravel()]))[c_offset:]
    mm.deviation_sample(to_dev(A), to_dev(B), dC, to_dev(D), m, n, k, nb, (ta, tb, fm.FP32, fm.FP32), stride, -3, h)
    same_hist(mm.read_deviation_hist(h), deviation_hist(A, B, C, D, ta, tb, stride, -3), shape)


@pytest.mark.parametrize("m,n", [(1, 4), (3, 5), (16, 16), (32, 32)])
@pytest.mark.parametrize("many", [False, True])
def test_truncating_variant_makes_zeros_positive(mm, m, n, many):
    """Both terms of the last sum negative and cut to zero: an exact zero, +0.0 (small tiles, tiled kernels, the scan kernel)."""
    half = lambda x: int(np.float16(x).view(np.uint16))
    nb, k = 3, 16 if m == 16 else 8
    A, B = np.zeros((nb, m, k), dtype=np.uint16), np.zeros((nb, n, k), dtype=np.uint16)
    A[..., -3], A[..., -2], A[..., -1] = half(1), half(-1 - 2.0 ** -10), half(2.0 ** -10)        # 1 - (1 + 2^-10) + (2^-10 - 2^-21)
    B[..., -3], B[..., -2], B[..., -1] = half(1), half(1), half(1 - 2.0 ** -11)
    C = np.resize(np.array([0x80000000, 0xB0000000, 0x80000001, 0, 0x30000000, 0xBF800000], dtype=np.uint32), (nb, m, n))
    p = TRZ.with_(group_len=8, frac_bits=23, frac_bits2=11)
    want = o2lib.emulate_mma(p, A, B, C, fm.FP16, fm.FP16)[0]
    assert (want == 0).any() and not (want == 0x80000000).any()
    if many and m == n:
        from test_gpu_many import run_many
        _, D, kern, _ = run_many(mm, [p, p.with_(frac_bits2=12)], A, B, C, fm.FP16, fm.FP16, ref=want)
        assert kern.startswith("multi x2"), kern
        assert_same(D[0], want, (m, n))
    else:
        assert_same(gpu_emulate(mm, p, A, B, C, fm.FP16, fm.FP16), want, (m, n))


@pytest.mark.parametrize("ta,tb,n,k", [(fm.FP16, fm.FP16, 8, 8), (fm.E4M3, fm.E5M2, 4, 40), (fm.E5M2, fm.FP16, 12, 17), (fm.FP16, fm.FP16, 4, 8192)])
def test_deviation_sample_four_outputs_per_thread(mm, ta, tb, n, k):
    """Enough outputs for four per thread: the oracle's histogram of one problem, many times over; one output per thread (an
    accumulator that is not 16-byte aligned) counts the same."""
    import torch
    rng = np.random.default_rng(60 + k)
    nb, m = 3, 5
    A, B = synth.random_bits(rng, (nb, m, k), ta), synth.random_bits(rng, (nb, n, k), tb)
    A[0, 0, 1] = synth.SPECIAL_CODES[ta][0]
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 100, 140)
    D = o2lib.emulate_mma(ModelParams(group_len=k, frac_bits=14), A, B, C, ta, tb)[0]
    # many problems; of long rows, one many times as high and wide
    reps = (1, 120, 240) if k == 8192 else ((1 << 19) // (nb * m * n) + 1, 1, 1)
    copies = reps[0] * reps[1] * reps[2]
    want = deviation_hist(A, B, C, D, ta, tb, 1, -6)
    want = {key: [v * copies for v in x] if key == "bins" else x * copies for key, x in want.items()}
    A, B, C, D = np.tile(A, (reps[0], reps[1], 1)), np.tile(B, (reps[0], reps[2], 1)), np.tile(C, reps), np.tile(D, reps)
    nb, m, n = D.shape
    for offset in (0, 1):
        dC = to_dev(np.concatenate([np.zeros(offset, np.uint32), C.ravel()]))[offset:]
        h = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
        mm.deviation_hist_reset(h)
        mm.deviation_sample(to_dev(A), to_dev(B), dC, to_dev(D), m, n, k, nb, (ta, tb, fm.FP32, fm.FP32), 1, -6, h)
        same_hist(mm.read_deviation_hist(h), want, (offset, k))


@pytest.mark.parametrize("ta,tb,m,n,k,stride,with_c,exps", [
    (fm.FP16, fm.FP16, 16, 16, 8, 1, True, (0, 30)), (fm.FP16, fm.FP16, 32, 32, 8, 3, True, (12, 22)), (fm.FP16, fm.FP16, 16, 32, 8, 4, True, (0, 30)),
    (fm.FP16, fm.FP16, 48, 16, 32, 1, False, (9, 24)), (fm.FP16, fm.FP16, 16, 64, 16, 2, True, (14, 20)), (fm.FP16, fm.FP16, 16, 32, 24, 1, True, (0, 30)),
    (fm.E4M3, fm.E4M3, 16, 16, 32, 1, True, (0, 14)), (fm.E4M3, fm.E5M2, 16, 96, 24, 1, True, (0, 14)), (fm.E5M2, fm.E4M3, 32, 32, 8, 4, False, (0, 14)),
    (fm.E5M2, fm.E5M2, 16, 32, 16, 1, True, (0, 30))])
@pytest.mark.parametrize("special", [False, True])
def test_deviation_sample_whole_tiles(mm, ta, tb, m, n, k, stride, with_c, exps, special):
    """The sums on the matrix cores: exponents that an exact chain holds and that it does not, outputs that leave its short end (a D far
    from the sum, accumulators far below it), infinities and NaN, strides; the oracle's histogram of a few tiles, many times over."""
    import torch
    rng = np.random.default_rng(90 + k + m + n + stride)
    nb = 3 if stride == 3 else 2
    A, B = synth.narrow_exponent_bits(rng, (nb, m, k), ta, *exps), synth.narrow_exponent_bits(rng, (nb, n, k), tb, *exps)
    A[0, 1], B[1, 2] = 0, 0
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 118, 132)
    C[rng.random(C.shape) < 0.02] = 0x00000003
    D = o2lib.emulate_mma(ModelParams(group_len=k, frac_bits=14), A, B, C if with_c else np.zeros_like(C), ta, tb)[0]
    D[0, 3, :6] = [0x00000001, 0x80000000, 0x00000000, 0x80800000, 0x3F800001, 0xBF800001]
    if special:
        D[0, 4, :2] = [0x7F7FFFFF, 0x5F000000]                       # (of one sign: their sum is the histogram's)
        A, B = synth.sprinkle(rng, A, synth.SPECIAL_CODES[ta], 0.01), synth.sprinkle(rng, B, synth.SPECIAL_CODES[tb], 0.01)
        C, D = (synth.sprinkle(rng, x, [0x7F800000, 0xFF800000, 0x7FC00000, 0xFFFFFFFF], 0.02) for x in (C, D))
    assert nb * m * n % stride == 0
    want = deviation_hist(A, B, C if with_c else None, D, ta, tb, stride, -5)
    copies = (1 << 17) // (nb * m * n) + 1
    want = {key: [v * copies for v in x] if key == "bins" else x * copies for key, x in want.items()}
    A, B, C, D = (np.tile(x, (copies, 1, 1)) for x in (A, B, C, D))
    same_hist(dev_hist(mm, A, B, C if with_c else None, D, ta, tb, stride, -5), want, (ta, tb, m, n, k, stride, special))


WHOLE_TILES = [(fm.FP16, fm.FP16, 32, 32, 8, 1, 2100), (fm.FP16, fm.FP16, 32, 32, 8, 3, 2100), (fm.FP16, fm.FP16, 16, 16, 8, 4, 4500),
               (fm.FP16, fm.FP16, 48, 16, 16, 1, 1400), (fm.E4M3, fm.E5M2, 16, 32, 24, 1, 4300), (fm.E5M2, fm.E5M2, 16, 16, 32, 1, 4200),
               (fm.E4M3, fm.E4M3, 32, 64, 8, 2, 1100), (fm.FP16, fm.FP16, 32, 32, 40, 1, 1100), (fm.FP16, fm.FP16, 16, 16, 64, 1, 4200),
               (fm.E4M3, fm.E5M2, 32, 32, 64, 1, 1100), (fm.E5M2, fm.E5M2, 48, 16, 56, 1, 1400)]


@pytest.mark.parametrize("ta,tb,m,n,k,stride,nb", WHOLE_TILES)
@pytest.mark.parametrize("kind", ["ordinary", "C far above", "C of any exponent", "D far off", "operands and C of any exponent"])
def test_deviation_sample_whole_tiles_that_all_differ(mm, ta, tb, m, n, k, stride, nb, kind):
    """More items than wavefronts, every tile another one, among them outputs whose difference no binary64 number holds; against the
    kernel of one or four outputs per thread (which takes A an element further on), and the first tiles against the oracle."""
    rng = np.random.default_rng(1000 + 7 * m + n + k + stride + len(kind))
    exps = {fm.FP16: (11, 19), fm.E4M3: (4, 10), fm.E5M2: (11, 19)}
    wide = kind.startswith("operands")
    A, B = (synth.random_bits(rng, (nb, x, k), t) if wide else synth.narrow_exponent_bits(rng, (nb, x, k), t, *exps[t]) for x, t in ((m, ta), (n, tb)))
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, *((150, 160) if kind == "C far above" else (1, 254) if "any exponent" in kind else (118, 132)))
    D = gpu_emulate(mm, ModelParams(group_len=8, frac_bits=24, frac_bits2=31, c_mode=C_AFTER_RD), A, B, C, ta, tb)
    if kind == "D far off":
        D = synth.narrow_exponent_bits(rng, D.shape, fm.FP32, 100, 190)
    if stride != 3:
        A, C = synth.sprinkle(rng, A, synth.SPECIAL_CODES[ta], 0.001), synth.sprinkle(rng, C, [0x7F800000, 0xFFC00000, 0x80000000], 0.002)
    dA, dB, dC, dD = (to_dev(x) for x in (A, B, C, D))
    shifted = to_dev(np.concatenate([np.zeros(1, A.dtype), A.ravel()]))[1:]
    dt = (ta, tb, fm.FP32, fm.FP32)
    import torch
    hists = []
    for a, name in ((dA, "whole tiles"), (shifted, "four outputs per thread" if stride == 1 else "one output per thread, split sum")):
        assert mm.deviation_sample_kernel(a, dB, dC, dD, m, n, k, nb, dt, stride) == name
        h = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
        mm.deviation_hist_reset(h)
        mm.deviation_sample(a, dB, dC, dD, m, n, k, nb, dt, stride, -5, h)
        hists.append(mm.read_deviation_hist(h))
    got, want = hists
    for key in ("n_samples", "n_skipped", "n_negative", "n_zero", "n_positive", "bins"):
        assert got[key] == want[key], (key, got[key], want[key])
    # every sum is a tree of fewer than 2^22 additions of values rounded once
    for key, scale in (("sum", "sum_abs"), ("sum_abs", "sum_abs"), ("sum_sq", "sum_sq")):
        assert abs(got[key] - want[key]) <= 2.0 ** (23 - 53) * want[scale], (key, got[key], want[key])
    t = 2 if stride < 3 else 12
    few = dev_hist(mm, A[:t], B[:t], C[:t], D[:t], ta, tb, stride, -5)
    exact = deviation_hist(A[:t], B[:t], C[:t], D[:t], ta, tb, stride, -5)
    for key in ("n_samples", "n_skipped", "n_negative", "n_zero", "n_positive", "bins"):
        assert few[key] == exact[key], (key, few[key], exact[key])


@pytest.mark.parametrize("lo,hi,tiles", [(118, 132, 1 << 14), (155, 160, 1 << 14), (1, 254, 1 << 10), (1, 254, 128)])
def test_whole_tiles_are_no_slower_for_any_accumulator(mm, lo, hi, tiles):
    """Accumulators of the products' size, 2^30 and of any exponent: as fast as the kernel that takes a call whose operands are not
    4-byte aligned (differences that no binary64 number holds took 1.9 to 5 times as long, each lane settling its own)."""
    import torch
    m, k = 32, 8
    dt = (fm.FP16, fm.FP16, fm.FP32, fm.FP32)
    A, B, D = (torch.empty(tiles * n + 2, dtype=t, device="cuda") for n, t in ((m * k, torch.int16), (m * k, torch.int16), (m * m, torch.int32)))
    C = torch.empty(tiles * m * m, dtype=torch.int32, device="cuda")
    for x, op in ((A, 0), (B, 1)):
        mm.generate(x, mm.FP16, m * k, 0, tiles, mm.GEN_UNIFORM_EXP, seed=3, operand=op, exp_lo=11, exp_hi=19)
    mm.generate(C, mm.FP32, m * m, 0, tiles, mm.GEN_UNIFORM_EXP, seed=3, operand=2, exp_lo=lo, exp_hi=hi)
    h = mm.model_create(group_len=8, frac_bits=24, frac_bits2=31, c_mode=mm.C_AFTER_RD)
    mm.emulate_mma(h, A, B, C, D, m, m, k, tiles, dt)
    mm.model_destroy(h)
    hist = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
    mm.deviation_hist_reset(hist)
    best = []
    for offset in (1, 0):
        times = []
        for _ in range(12):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                mm.deviation_sample(A[offset:], B, C, D, m, m, k, tiles, dt, 1, -5, hist)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        best.append(min(times))
    assert best[1] < 1.1 * best[0], best


@pytest.mark.parametrize("stride", [(1 << 61) + 1, 1 << 61, 1 << 63, (1 << 32) + 1, (1 << 64) - 1, (1 << 64) - (513 << 8)])
def test_deviation_sample_strides_beyond_the_outputs(mm, stride):
    """One sample, output 0, also where the product of stride and k, or the sum of stride and outputs, leaves 64 bits."""
    rng = np.random.default_rng(17)
    nb, m, n, k = 513, 16, 16, 8
    A, B = synth.narrow_exponent_bits(rng, (nb, m, k), fm.FP16, 10, 20), synth.narrow_exponent_bits(rng, (nb, n, k), fm.FP16, 10, 20)
    C = synth.narrow_exponent_bits(rng, (nb, m, n), fm.FP32, 118, 132)
    got = dev_hist(mm, A, B, C, C, fm.FP16, fm.FP16, stride, -5)
    same_hist(got, deviation_hist(A[:1], B[:1], C[:1], C[:1], fm.FP16, fm.FP16, 256, -5), stride)
    assert got["n_samples"] == 1


def test_few_outputs_with_long_rows_keep_one_per_thread(mm):
    """4096 outputs of 4096 terms: as fast as the call whose accumulator is not 16-byte aligned, which always runs one output
    per thread (four per thread took 2.6 times as long)."""
    import torch
    m, k = 64, 4096
    z = torch.zeros(m * k, dtype=torch.int16, device="cuda")
    C = torch.zeros(m * m + 4, dtype=torch.int32, device="cuda")
    h = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
    mm.deviation_hist_reset(h)
    best = []
    for offset in (1, 0):
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            mm.deviation_sample(z, z, C[offset:], C, m, m, k, 1, (fm.FP16, fm.FP16, fm.FP32, fm.FP32), 1, 0, h)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        best.append(min(times))
    assert best[1] < 1.6 * best[0], best


@pytest.mark.parametrize("sign", [1, -1])
def test_deviation_sample_residue_of_the_lower_sum(mm, sign):
    """D so large that the low half of the pair cannot hold both sums, and an accumulator of the size of what is left over, of
    either sign: products 2^39 in all and one of 2^-40, c = +-2^-40, D from 2^44 to +-2^98."""
    k = 1032
    A, B = np.zeros((1, 4, k), dtype=np.uint16), np.zeros((1, 4, k), dtype=np.uint16)
    A[..., :1024], B[..., :1024] = 29 << 10, 30 << 10                   # 2^14 times 2^15
    A[..., 1024], B[..., 1024] = 0x0010, 0x0010                         # 2^-20 each
    C = np.full((1, 4, 4), (87 << 23) | (0x80000000 if sign < 0 else 0), dtype=np.uint32)         # +-2^-40
    D = np.full((1, 4, 4), (127 + 98) << 23, dtype=np.uint32)
    D[0, 1], D[0, 2], D[0, 3] = (127 + 93) << 23, ((127 + 98) << 23) | 0x80000000, (127 + 44) << 23
    for bin_exp in (98, 60, 44, -40):
        h = dev_hist(mm, A, B, C, D, fm.FP16, fm.FP16, 1, bin_exp)
        same_hist(h, deviation_hist(A, B, C, D, fm.FP16, fm.FP16, 1, bin_exp), (sign, bin_exp))


def test_deviation_sample_extremes_and_errors(mm):
    import torch
    # the widest reach of the exact sum: BF16 products at both ends of the range next to binary32's smallest subnormal
    big, tiny = 0x7F7F, 0x0001
    A = np.array([[[big, tiny, big, tiny]]], dtype=np.uint16)
    B = np.array([[[big, tiny, 0xFF7F, 0x8001]]], dtype=np.uint16)         # everything cancels
    C = np.array([[[0x00000001]]], dtype=np.uint32)
    D = np.array([[[0x00000001]]], dtype=np.uint32)
    h = dev_hist(mm, A, B, C, D, fm.BF16, fm.BF16, 1, -149)
    assert h["n_zero"] == 1 and h["bins"][32] == 1
    same_hist(h, deviation_hist(A, B, C, D, fm.BF16, fm.BF16, 1, -149), "cancelling extremes")
    D[0, 0, 0] = 0x7F7FFFFF
    h = dev_hist(mm, A[:, :, :2], B[:, :, :2], C, D, fm.BF16, fm.BF16, 1, 250)
    same_hist(h, deviation_hist(A[:, :, :2], B[:, :, :2], C, D, fm.BF16, fm.BF16, 1, 250), "largest product")
    z = torch.zeros(64, dtype=torch.int32, device="cuda")
    hist = torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda")
    for kw, status in ((dict(stride=0), 3), (dict(bin_exp=-281), 1), (dict(dtypes=(mm.FP32, mm.FP32, mm.FP32, mm.FP32)), 2), (dict(k=0), 3)):
        args = dict(m=2, n=2, k=4, batch=1, dtypes=(mm.FP16, mm.FP16, mm.FP32, mm.FP32), stride=1, bin_exp=0)
        args.update(kw)
        with pytest.raises(mm.MmaemuError) as ei:
            mm.deviation_sample(z, z, z, z, args["m"], args["n"], args["k"], args["batch"], args["dtypes"], args["stride"], args["bin_exp"], hist)
        assert ei.value.status == status, kw


def test_bias_experiment_workload(mm):
    from paper_2511_10909_amd import configs
    nt, chunk = 1 << 16, 1 << 14
    r = configs.bias_experiment(n_tiles=nt, chunk=chunk, seed=2, stride=1, keep_first_chunk=True)
    assert r["kernels"]["rd"].startswith("tiled") and r["kernels"]["rz"].startswith("tiled")
    H = r["hists"]
    n = nt * 1024
    for name in ("rd", "rz", "mfma"):
        h = H[name]
        assert h["n_samples"] == n and h["n_skipped"] == 0 and sum(h["bins"]) == n
        assert h["n_negative"] + h["n_zero"] + h["n_positive"] == n
    mean = {k: h["sum"] / n for k, h in H.items()}
    sd_of_mean = {k: (h["sum_sq"] / n - mean[k] ** 2) ** 0.5 / n ** 0.5 for k, h in H.items()}
    assert mean["rd"] < -50 * sd_of_mean["rd"]                    # Sec. 6.2.4: shifted toward the negative side
    assert abs(mean["rz"]) < 5 * sd_of_mean["rz"]                 # the truncating variant is centred
    assert H["rd"]["n_negative"] > 1.2 * H["rd"]["n_positive"] and 0.98 < H["rz"]["n_negative"] / H["rz"]["n_positive"] < 1.02
    assert mean["mfma"] < -50 * sd_of_mean["mfma"]                # this GPU's FP16 instruction rounds down as well
    # a prefix against the oracle: generated inputs, both variants' outputs, and the histogram of that prefix
    f = r["first"]
    t = 3
    A = to_host(f["A"], np.uint16)[:t]; B = to_host(f["B"], np.uint16)[:t]; C = to_host(f["C"], np.uint32)[:t]
    gp = lambda op, **kw: ogen.GenParams(family=ogen.GEN_NORMAL, seed=2, operand=op, **kw)
    assert np.array_equal(A.ravel(), ogen.generate(gp(0, scale_scope=ogen.SCALE_FACTOR, scale_target=1000.0), fm.FP16, 256, 0, t).ravel())
    assert np.array_equal(C.ravel(), ogen.generate(gp(2), fm.FP32, 1024, 0, t).ravel())
    base = ModelParams(group_len=8, frac_bits=24, frac_bits2=31, c_mode=C_AFTER_RD)
    jobs = [(dataclasses.asdict(base.with_(rd_toward_zero=z)), A, B, C, fm.FP16, fm.FP16, None, None, 0) for z in (False, True)]
    for name, want in zip(("rd", "rz"), run_pool(jobs, workers=2)):
        got = to_host(f[name], np.uint32)[:t]
        assert np.array_equal(got, want), name
        hist = deviation_hist(A, B, C, want, fm.FP16, fm.FP16, 1, configs.BIAS_BIN_EXP)
        same_hist(dev_hist(mm, A, B, C, got, fm.FP16, fm.FP16, 1, configs.BIAS_BIN_EXP), hist, name)
        # ... and that prefix many times over, in the kernel for whole tiles, which fills the workload's histograms
        copies = 50
        many = [np.tile(x, (copies, 1, 1)) for x in (A, B, C, got)]
        assert mm.deviation_sample_kernel(4096, 4096, 4096, 4096, 32, 32, 8, t * copies, (fm.FP16, fm.FP16, fm.FP32, fm.FP32), 1) == "whole tiles"
        same_hist(dev_hist(mm, *many, fm.FP16, fm.FP16, 1, configs.BIAS_BIN_EXP),
                  {key: [v * copies for v in x] if key == "bins" else x * copies for key, x in hist.items()}, name)

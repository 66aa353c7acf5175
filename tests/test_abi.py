"""The C-ABI library loads without a GPU and exports every function the public header declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mmaemu.h")
LIB = os.path.join(ROOT, "paper_2511_10909_amd", "libmmaemu.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2511_10909_amd.build import build_library
        build_library(verbose=False)
    return ctypes.CDLL(LIB)


def declared_functions():
    with open(HEADER) as fh:
        text = fh.read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mmaemu_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_boundary():
    names = declared_functions()
    for required in ("mmaemu_model_create", "mmaemu_model_destroy", "mmaemu_emulate_mma", "mmaemu_compare",
                     "mmaemu_stats_reset", "mmaemu_generate", "mmaemu_mfma_probe", "mmaemu_exact_dot_sample",
                     "mmaemu_status_string", "mmaemu_last_error"):
        assert required in names


def test_every_declared_symbol_is_exported(lib):
    for name in declared_functions():
        assert hasattr(lib, name), name


def test_struct_sizes_match_binding():
    from paper_2511_10909_amd import binding as mm
    assert ctypes.sizeof(mm.ModelParams) == 100
    assert ctypes.sizeof(mm.DeviationHist) == 8 * 72
    assert ctypes.sizeof(mm.Stats) == 8 * 39
    assert ctypes.sizeof(mm.ErrStats) == 8 * 44
    assert ctypes.sizeof(mm.GenParams) == 48


def test_host_side_validation_needs_no_gpu():
    from paper_2511_10909_amd import binding as mm
    h = mm.model_create(group_len=8, frac_bits=24)
    assert mm.model_get_params(h)["group_len"] == 8
    mm.model_destroy(h)
    mm.model_destroy(None)
    for kw, status in ((dict(frac_bits=49), 2), (dict(frac_bits=41, frac_bits2=31, c_mode=2), 2), (dict(out_round=2), 1), (dict(c_mode=5), 1), (dict(align_round=1), 2),
                       (dict(out_mant_bits=13), 2), (dict(out_mant_bits=10, out_round=1), 2), (dict(frac_bits2=31), 2), (dict(c_mode=2, frac_bits2=49), 2), (dict(split=1), 2), (dict(c_mode=2, split=4), 1),
                       (dict(c_mode=3, frac_bits2=31, frac_bits_acc=24), 2), (dict(c_mode=2, frac_bits_merge=24), 2), (dict(skip_zero_terms=2), 1), (dict(family=4), 1), (dict(family=2), 2), (dict(family=1, group_len=8), 2), (dict(family=1, group_len=4, ftz_out=True), 2), (dict(struct_size=40), 1),
                       (dict(rd_toward_zero=True), 2), (dict(c_mode=2, frac_bits2=31, rd_toward_zero=2), 2), (dict(group_len=(1 << 20) + 1), 2)):
        with pytest.raises(mm.MmaemuError) as ei:
            mm.model_create(**kw)
        assert ei.value.status == status, kw
    assert "frac_bits" in mm.last_error() or "group_len" in mm.last_error()
    mm.model_destroy(mm.model_create(group_len=16, frac_bits=13, out_round=mm.RZ, out_mant_bits=13))
    for mode in (mm.C_AFTER_RD, mm.C_AFTER_RD_EVEN_ODD):
        h = mm.model_create(group_len=8, frac_bits=24, frac_bits2=31, c_mode=mode)
        assert mm.model_get_params(h)["frac_bits2"] == 31
        mm.model_destroy(h)
    info = mm.mfma_info(mm.MFMA_F32_16X16X32_FP8_BF8)
    assert info == dict(m=16, n=16, k=32, a=mm.E4M3, b=mm.E5M2)
    with pytest.raises(mm.MmaemuError):
        mm.mfma_info(99)


def test_emulate_rejects_bad_arguments_before_any_gpu_call():
    """Every check of mmaemu_emulate_mma's arguments runs on the host: fake addresses never reach a kernel."""
    from paper_2511_10909_amd import binding as mm
    h = mm.model_create(group_len=8, frac_bits=24)
    dt = (mm.FP16, mm.FP16, mm.FP32, mm.FP32)
    ok = 0x1000
    cases = [
        (dict(A=ok + 1), 1),          # FP16 operand at an odd address
        (dict(C=ok + 2), 1),          # FP32 accumulator off a 4-byte boundary
        (dict(D=ok + 1), 1),
        (dict(A=None), 1),
        (dict(k=12), 3),              # k is not a multiple of the group length
        (dict(m=0), 3),
        (dict(k=(1 << 20) + 8), 3),
    ]
    for change, status in cases:
        a = dict(A=ok, B=ok, C=ok, D=ok, m=16, n=16, k=16, batch=1)
        a.update(change)
        with pytest.raises(mm.MmaemuError) as ei:
            mm.emulate_mma(h, a["A"], a["B"], a["C"], a["D"], a["m"], a["n"], a["k"], a["batch"], dt, stream=0)
        assert ei.value.status == status, (change, mm.last_error())
    # batch = 0 is a no-op whatever the pointers are
    mm.emulate_mma(h, None, None, None, None, 16, 16, 16, 0, dt, stream=0)
    with pytest.raises(mm.MmaemuError) as ei:
        mm.emulate_mma(h, ok, ok, ok, ok, 16, 16, 16, 1, (mm.TF32, mm.FP16, mm.FP32, mm.FP32), stream=0)
    assert ei.value.status == 2
    mm.model_destroy(h)


def test_fma_family_argument_checks():
    from paper_2511_10909_amd import binding as mm
    for kw in (dict(group_len=2), dict(ftz_in=True), dict(out_round=mm.RZ), dict(c_mode=mm.C_AFTER_EXACT), dict(out_mant_bits=13, out_round=mm.RZ)):
        with pytest.raises(mm.MmaemuError) as ei:
            mm.model_create(family=mm.FAMILY_FMA, **kw)
        assert ei.value.status == 2, kw
    h = mm.model_create(family=mm.FAMILY_FMA, group_len=1)
    ok = 0x1000
    for dt in ((mm.BF16, mm.BF16, mm.FP32, mm.FP32), (mm.TF32, mm.TF32, mm.FP32, mm.FP32), (mm.FP32, mm.FP32, mm.FP16, mm.FP16)):
        with pytest.raises(mm.MmaemuError) as ei:
            mm.emulate_mma(h, ok, ok, ok, ok, 16, 16, 4, 1, dt, stream=0)
        assert ei.value.status == 2, dt
    with pytest.raises(mm.MmaemuError):
        mm.emulate_mma_scaled(h, ok, ok, ok, ok, ok, ok, 4, 16, 16, 4, 1, (mm.FP32,) * 4, stream=0)
    mm.emulate_mma(h, None, None, None, None, 16, 16, 4, 0, (mm.FP32,) * 4, stream=0)     # batch = 0: no-op
    mm.model_destroy(h)


def test_compare_many_classes_is_a_host_side_query():
    """Which models mmaemu_emulate_compare_many runs in common launches: decided on the host, no GPU needed."""
    from paper_2511_10909_amd import binding as mm
    rd = dict(group_len=8, frac_bits=24, frac_bits2=31, c_mode=mm.C_AFTER_RD)
    sets = [dict(group_len=8, frac_bits=24), dict(group_len=16, frac_bits=32, out_round=mm.RZ, ftz_in=True),      # T-FDPA: class 0
            rd, dict(rd, f2_at_leading_bit=True, sum_drop_distance=28, acc_special_truncation=True),               # TR-FDPA: class 1
            dict(rd, skip_zero_terms=True), dict(rd, skip_zero_terms=True, ftz_in=True),                           # zero terms out of the maxima: 2, 3
            dict(rd, split=mm.SPLIT_HALVES),                                                                       # halves / quarters: 4 to 6
            dict(group_len=8, frac_bits=24, c_mode=mm.C_AFTER_EXACT), dict(rd, split=mm.SPLIT_EVEN_ODD),           # not in the scan kernel; even / odd: 7 to 9
            dict(group_len=2, frac_bits=24), dict(group_len=8, frac_bits=44)]
    hs = [mm.model_create(**kw) for kw in sets]
    dt = (mm.FP16, mm.FP16, mm.FP32, mm.FP32)
    assert mm.compare_many_classes(hs, 16, 16, 16, dt) == [0, 0, 1, 1, 2, 3, 4, -1, 7, -1, -1]
    assert mm.compare_many_classes(hs[:6], 32, 32, 16, dt) == [0, 0, 1, 1, 2, 3]
    assert mm.compare_many_classes(hs[:6], 16, 16, 32, (mm.BF16, mm.BF16, mm.FP32, mm.FP32)) == [0, 0, 1, 1, 2, 3]
    assert mm.compare_many_classes(hs[:3], 16, 16, 64, dt) == [-1, -1, -1]          # shapes the kernel does not stage whole
    assert mm.compare_many_classes(hs[:3], 20, 20, 16, dt) == [-1, -1, -1]
    assert mm.compare_many_classes(hs[:3], 16, 16, 16, (mm.TF32, mm.TF32, mm.FP32, mm.FP32)) == [-1, -1, -1]
    wide = mm.model_create(**dict(rd, wide_products=True))
    assert mm.compare_many_classes([wide], 16, 16, 16, (mm.BF16, mm.BF16, mm.FP32, mm.FP32)) == [-1]
    assert mm.compare_many_classes([wide], 16, 16, 16, dt) == [1]
    quarters = [mm.model_create(**dict(rd, group_len=16, frac_bits=13, split=mm.SPLIT_QUARTERS, skip_zero_terms=True, ftz_in=f)) for f in (False, True)]
    assert mm.compare_many_classes(quarters, 16, 16, 32, (mm.E4M3, mm.E5M2, mm.FP32, mm.FP32)) == [5, 6]
    assert mm.compare_many_classes(quarters, 16, 16, 32, (mm.BF16, mm.BF16, mm.FP32, mm.FP32)) == [-1, -1]     # (binary32 values only)
    assert mm.compare_many_classes(quarters, 32, 32, 8, dt) == [-1, -1]                                         # (the group is the whole k = 8: no quarters of four)
    for h in quarters:
        mm.model_destroy(h)
    for h in hs + [wide]:
        mm.model_destroy(h)


def test_deviation_sample_takes_up_to_2_43_samples():
    """The limit of the 32-bit counters of a workgroup, decided before anything is launched; without a GPU the largest
    accepted call ends in a HIP error, not in a refusal of its shape."""
    import torch
    from paper_2511_10909_amd import binding as mm
    if torch.cuda.is_available():
        pytest.skip("the accepted call must not reach a device")
    call = lambda batch: mm.deviation_sample(4096, 4096, 4096, 4096, 1, 1, 8, batch, (mm.FP16, mm.FP16, mm.FP32, mm.FP32), 1, 0, 4096, stream=0)
    for batch, status in (((1 << 43) + 1, 3), (1 << 43, 4), (1 << 42, 4)):
        with pytest.raises(mm.MmaemuError) as ei:
            call(batch)
        assert ei.value.status == status, (batch, str(ei.value))


def test_deviation_sample_limit_holds_for_whole_tiles():
    """The same limit where the kernel for whole tiles would take the call; the refusal comes before any launch."""
    import torch
    from paper_2511_10909_amd import binding as mm
    call = lambda m, n, k, batch, stride: mm.deviation_sample(4096, 4096, 4096, 4096, m, n, k, batch, (mm.FP16, mm.FP16, mm.FP32, mm.FP32), stride, 0, 4096, stream=0)
    shapes = [(16, 16, 8, (1 << 43) // 256 + 1, 1), (32, 32, 32, 1 << 34, 1), (16, 16, 8, 1 << 38, 4), (16, 16, 8, 1 << 54, 2)]
    accepted = [(16, 16, 8, (1 << 43) // 256, 1), (16, 16, 8, 1 << 37, 4)]
    for args in shapes + ([] if torch.cuda.is_available() else accepted):          # (an accepted call must not reach a device: without one it is a HIP error)
        with pytest.raises(mm.MmaemuError) as ei:
            call(*args)
        assert ei.value.status == (3 if args in shapes else 4), (args, str(ei.value))


def test_deviation_sample_kernel_for_a_call():
    """Each side of every condition on the kernel for whole tiles, strides whose product with k leaves 64 bits among them."""
    from paper_2511_10909_amd import binding as mm
    base = dict(A=4096, B=4096, C=4096, D=4096, m=32, n=32, k=8, batch=128, a=mm.FP16, b=mm.FP16, stride=1)
    def kernel(**kw):
        c = dict(base, **kw)
        return mm.deviation_sample_kernel(c["A"], c["B"], c["C"], c["D"], c["m"], c["n"], c["k"], c["batch"], (c["a"], c["b"], mm.FP32, mm.FP32), c["stride"])
    for kw in ({}, dict(C=None), dict(stride=4), dict(k=32), dict(k=16, stride=2), dict(k=24), dict(A=4100, B=4108), dict(C=4104, D=4112), dict(n=16, m=64, C=4100, D=4108),
               dict(k=40, batch=1024), dict(k=64, batch=1024), dict(a=mm.E4M3, b=mm.E5M2), dict(m=16, n=16, batch=512), dict(m=48, n=48, batch=57)):
        assert kernel(**kw) == "whole tiles", kw
    one, four = "one output per thread, split sum", "four outputs per thread"
    for kw, want in ((dict(stride=5), one), (dict(stride=33), one), (dict(k=16, stride=3), one), (dict(k=32, stride=2), one), (dict(k=40), one), (dict(k=9), one),
                     (dict(batch=127), one), (dict(A=4098), one), (dict(B=4098), one), (dict(C=4100), one), (dict(D=4100), one), (dict(a=mm.E4M3, B=4097, b=mm.E4M3), one),
                     (dict(m=31, batch=133), one), (dict(n=36), one), (dict(a=mm.FP16, b=mm.E4M3), one), (dict(a=mm.E2M3, b=mm.E2M3), one),
                     (dict(a=mm.BF16, b=mm.BF16), "one output per thread, pairs"), (dict(k=40, batch=512), four), (dict(k=64, batch=1023), four), (dict(k=72, batch=1024), four), (dict(k=64, batch=2048, stride=2), one),
                     (dict(k=40, batch=2048, stride=2), one), (dict(k=64, batch=256), one),
                     (dict(n=1 << 25, m=16, batch=1), four), (dict(k=1 << 14), "one output per thread, pairs")):
        assert kernel(**kw) == want, kw
    for k in (8, 16, 24, 32, 40, 64):
        for stride in [(1 << 64) // k + d for d in range(4)] + [(1 << e) + d for e in (32, 59, 60, 61, 62, 63) for d in (0, 1, 2, 4)] + [(1 << 64) - (1 << 20)]:
            assert kernel(k=k, stride=stride) == one, (k, stride)
    for kw, status in ((dict(stride=0), 3), (dict(D=None), 1), (dict(A=4097), 1), (dict(a=mm.TF32), 2)):
        with pytest.raises(mm.MmaemuError) as ei:
            kernel(**kw)
        assert ei.value.status == status, kw


def test_current_stream_without_the_private_call(monkeypatch):
    """Both ways to the current stream's handle: torch's raw one for the current device, and the stream object's where torch lacks it."""
    import types
    import torch
    from paper_2511_10909_amd import binding as mm
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(mm, "_raw_stream", lambda device: 100 + device)
    assert mm._stream(None) == 103
    monkeypatch.setattr(mm, "_raw_stream", None)
    assert mm._stream(None) == 77 and mm._stream(5) == 5

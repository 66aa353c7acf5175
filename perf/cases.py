"""Measured cases: the work of randomized validation (Sec. 3.1, Step 4), through the library's entry points.

What a user of the library runs is loops of the same few calls: generate operand tiles, issue the native instruction on
them, evaluate one or many models, count differing outputs, and beside that evaluate a model on a GEMM-shaped problem or
collect the distribution of its deviations.  Each case is one pass of such a loop over one chunk of tiles, or one such
problem; the sizes are the repository's own workloads, tests and benchmark, and `draw` covers the ranges around them.

Bit patterns are returned as whole numbers (they are defined bit for bit and stay the same); where a pattern has a value
that plain 64-bit arithmetic approaches, the same buffer is also returned as binary32 and `exact` gives that value.
"""
import math

import torch

from paper_2511_10909_amd import binding as mm
from paper_2511_10909_amd import configs, presets

FP32_OUT = (mm.FP32, mm.FP32)
TYPES = {"bf16": mm.BF16, "fp16": mm.FP16, "tf32": mm.TF32, "fp32": mm.FP32}

# One candidate list of Step 4: the fitted 16-bit set of gfx950 among others of other widths and group lengths.
TR_SHAPES = {"16x16x16": (mm.MFMA_F32_16X16X16_F16, mm.MFMA_F32_16X16X16_BF16),
             "32x32x8": (mm.MFMA_F32_32X32X8_F16, mm.MFMA_F32_32X32X8_BF16),
             "16x16x32": (mm.MFMA_F32_16X16X32_F16, mm.MFMA_F32_16X16X32_BF16)}

# Instructions whose fitted models are checked over every input family.
INSTRUCTIONS = {
    "16x16x16_f16": mm.MFMA_F32_16X16X16_F16, "32x32x8_bf16": mm.MFMA_F32_32X32X8_BF16,
    "16x16x32_bf16": mm.MFMA_F32_16X16X32_BF16, "32x32x16_f16": mm.MFMA_F32_32X32X16_F16,
    "16x16x32_fp8_bf8": mm.MFMA_F32_16X16X32_FP8_BF8, "32x32x16_bf8_bf8": mm.MFMA_F32_32X32X16_BF8_BF8,
    "16x16x4_f32": mm.MFMA_F32_16X16X4_F32, "32x32x2_f32": mm.MFMA_F32_32X32X2_F32,
    "4x4x4_16b_f16": mm.MFMA_MULTIBLOCK_F16_IDS[2], "4x4x4_16b_bf16": mm.MFMA_MULTIBLOCK_BF16_IDS[2],
    "16x16x4_4b_f16": mm.MFMA_MULTIBLOCK_F16_IDS[1], "32x32x4_2b_bf16": mm.MFMA_MULTIBLOCK_BF16_IDS[0],
    "16x16x128_fp8_fp8": mm.mfma_scale_id(mm.E4M3, mm.E4M3), "16x16x128_fp4_fp4": mm.mfma_scale_id(mm.E2M1, mm.E2M1),
    "32x32x64_fp8_bf6": mm.mfma_scale_id(mm.E4M3, mm.E3M2, 32)}


def listed():
    return [
        # A probing step or a first look at a model: 64 tiles, two models compared, the instruction beside them.
        # Nine small launches: latency and host work.
        dict(name="check_fp16_64", kind="check", tiles=64),
        # The closed-loop scan, one chunk as the benchmark runs it: sixteen T-FDPA sets against the instruction, on
        # BF16 bit patterns (the whole exponent range) and on per-tile scaled FP8 values.
        dict(name="scan_bf16_64k", kind="scan", type="bf16", tiles=1 << 16),
        dict(name="scan_fp8_64k", kind="scan", type="fp8", tiles=1 << 16),
        # The same loop on sixteen TR-FDPA candidates (the model family of the CDNA instructions), N(0,1) operands.
        dict(name="candidates_tr_fp16", kind="candidates", type="fp16", shape="16x16x16", tiles=1 << 15),
        # The subnormal stress workload, one chunk: three flush variants against each other.
        dict(name="flush_fp16_256k", kind="flush", tiles=1 << 18),
        # GEMM-shaped problems: a chained against a fully fused model; a large FP8 one with exact dots on 1 % of it;
        # a ragged one in TF32.
        dict(name="gemm_bf16_1024", kind="gemm", type="bf16", m=1024, n=1024, k=1024),
        dict(name="gemm_fp8_4096", kind="gemm", type="fp8", m=4096, n=4096, k=4096),
        dict(name="gemm_tf32_ragged", kind="gemm", type="tf32", m=1000, n=744, k=512),
        # A fitted model against its instruction over every input family: FP8, block-scaled FP8, and the 4x4x4 blocks
        # (tiles far below a workgroup's size).
        dict(name="families_fp8_16x16x32", kind="families", instr="16x16x32_fp8_bf8", tiles=1 << 13),
        dict(name="families_scaled_fp8", kind="families", instr="16x16x128_fp8_fp8", tiles=1 << 11),
        dict(name="families_4x4x4_fp16", kind="families", instr="4x4x4_16b_f16", tiles=1 << 18),
        # The numerical-bias experiment of Sec. 6.2.4, one chunk: two models and the instruction, every output's
        # deviation from its exact result.
        dict(name="bias_fp16_16k", kind="bias", tiles=1 << 14, stride=1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["check", "scan", "candidates", "flush", "gemm", "gemm", "families", "families", "bias"])
    if kind == "check":
        return dict(kind=kind, tiles=_log_int(rng, 1, 10000))
    if kind == "scan":
        return dict(kind=kind, type=rng.choice(["bf16", "fp8"]), tiles=_log_int(rng, 500, 1 << 16))
    if kind == "candidates":
        return dict(kind=kind, type=rng.choice(["fp16", "bf16"]), shape=rng.choice(sorted(TR_SHAPES)), tiles=_log_int(rng, 500, 1 << 14))
    if kind == "flush":
        return dict(kind=kind, tiles=_log_int(rng, 500, 1 << 18))
    if kind == "gemm":
        t = rng.choice(["bf16", "fp8", "tf32", "fp16", "fp32"])
        top = 4096 if t in ("fp8", "fp32") else 1100
        return dict(kind=kind, type=t, m=_log_int(rng, 40, top), n=_log_int(rng, 40, top), k=32 * _log_int(rng, 2, top // 32))
    if kind == "families":
        instr = rng.choice(sorted(INSTRUCTIONS))
        info = mm.mfma_info(INSTRUCTIONS[instr])
        most = (1 << 26) // (info["m"] * info["n"] * max(4, info["k"]))
        return dict(kind=kind, instr=instr, tiles=_log_int(rng, 200, max(2000, most)))
    return dict(kind=kind, tiles=_log_int(rng, 200, 1 << 14), stride=rng.randint(1, 7))


# ---- operands of the GEMM-shaped problems ---------------------------------------------------------------------------

def _gemm_operands(case, seed):
    """(A, B, C) as values a product computes with, and the types of A and B."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    m, n, k, t = case["m"], case["n"], case["k"], case["type"]
    a, b = torch.randn((m, k), generator=g, device="cuda"), torch.randn((n, k), generator=g, device="cuda")
    c = torch.zeros((m, n), device="cuda") if t in ("bf16", "fp8") else torch.randn((m, n), generator=g, device="cuda")
    if t == "fp8":
        a = (a * (448.0 / a.abs().max())).to(torch.float8_e4m3fn)
        b = (b * (57344.0 / b.abs().max())).to(torch.float8_e5m2)
        return a, b, c, mm.E4M3, mm.E5M2
    if t in ("bf16", "fp16"):
        dt = torch.bfloat16 if t == "bf16" else torch.float16
        return a.to(dt), b.to(dt), c, TYPES[t], TYPES[t]
    if t == "tf32":                                             # ten mantissa bits of a binary32 word
        a, b = ((x.view(torch.int32) & -8192).view(torch.float32) for x in (a, b))
    return a, b, c, TYPES[t], TYPES[t]


def _gemm_models(t):
    if t == "bf16":                                             # groups of eight added to the running sum, against one fused sum
        return [dict(group_len=8, frac_bits=24, c_mode=mm.C_AFTER_EXACT), dict(group_len=0, frac_bits=24, c_mode=mm.C_IN_GROUP)]
    if t == "fp8":
        return [dict(group_len=32, frac_bits=14, out_round=mm.RNE)]
    if t == "tf32":
        return [presets.PAPER[("hopper", "tf32")]]
    if t == "fp16":
        return [presets.PAPER[("cdna3", "fp16")]]
    return [presets.PAPER[("fma", "fp32")]]


def _as_float(x):
    return x.view(torch.float32)


def _new(shape, dtype_id):
    return torch.empty(shape, dtype={1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[mm.ELEM_BYTES[dtype_id]], device="cuda")


def _stats(count):
    st = torch.empty(count * mm.STATS_BYTES, dtype=torch.uint8, device="cuda")
    for i in range(count):
        mm.stats_reset(st[i * mm.STATS_BYTES:])
    return st


def _families(instr):
    info = mm.mfma_info(instr)
    return configs.validation_families(info["a"], info["b"])


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=seed)
    if kind == "check":
        nt = case["tiles"]
        s["A"], s["B"] = _new((nt, 16, 16), mm.FP16), _new((nt, 16, 16), mm.FP16)
        s["C"], s["D0"], s["D1"], s["Dhw"] = (_new((nt, 16, 16), mm.FP32) for _ in range(4))
        s["stats"] = _stats(1)
        s["models"] = [mm.model_create(group_len=16, frac_bits=27, out_round=r) for r in (mm.RNE, mm.RZ)]
    elif kind == "scan":
        s["scan"] = configs.ClosedLoopScan(case["type"], case["tiles"], seed)
    elif kind == "candidates":
        instr = TR_SHAPES[case["shape"]][case["type"] == "bf16"]
        info, nt = mm.mfma_info(instr), case["tiles"]
        fitted = presets.GFX950_MFMA[instr]
        sets = [dict(fitted, frac_bits=F, frac_bits2=F2, group_len=L) for F in (20, 24) for F2 in (27, 31) for L in (4, 8, min(16, info["k"]), 8)]
        sets[15] = dict(fitted)
        s.update(instr=instr, info=info, models=[mm.model_create(**p) for p in sets], stats=_stats(16))
        s["A"], s["B"] = _new((nt, info["m"], info["k"]), info["a"]), _new((nt, info["n"], info["k"]), info["b"])
        s["C"], s["Dhw"] = _new((nt, info["m"], info["n"]), mm.FP32), _new((nt, info["m"], info["n"]), mm.FP32)
    elif kind == "flush":
        nt = case["tiles"]
        s["A"], s["B"], s["C"] = _new((nt, 32, 8), mm.FP16), _new((nt, 32, 8), mm.FP16), _new((nt, 32, 32), mm.FP32)
        s["models"] = [mm.model_create(group_len=8, frac_bits=24, out_round=mm.RNE, **kw) for _, kw in configs.CONFIG4_VARIANTS]
        s["stats"] = _stats(3)
    elif kind == "gemm":
        a, b, c, ta, tb = _gemm_operands(case, seed)
        s.update(A=a, B=b, C=c, dt=(ta, tb) + FP32_OUT, models=[mm.model_create(**p) for p in _gemm_models(case["type"])])
        s["D"] = [_new((case["m"], case["n"]), mm.FP32) for _ in s["models"]]
        s["stats"] = _stats(1)
        s["err"] = torch.empty(mm.ERR_STATS_BYTES, dtype=torch.uint8, device="cuda")
    elif kind == "families":
        instr = INSTRUCTIONS[case["instr"]]
        info, nt = mm.mfma_info(instr), case["tiles"]
        fams = _families(instr)
        s.update(instr=instr, info=info, fams=fams, scaled=case["instr"].startswith(("16x16x128", "32x32x64")),
                 model=mm.model_create(**presets.GFX950_MFMA[instr]), stats=_stats(len(fams)))
        s["A"], s["B"] = _new((nt, info["m"], info["k"]), info["a"]), _new((nt, info["n"], info["k"]), info["b"])
        s["C"], s["Dhw"], s["D"] = (_new((nt, info["m"], info["n"]), mm.FP32) for _ in range(3))
        if s["scaled"]:
            s["SA"], s["SB"] = _new((nt, info["m"], info["k"] // 32), mm.E8M0), _new((nt, info["n"], info["k"] // 32), mm.E8M0)
    else:
        nt = case["tiles"]
        s["A"], s["B"] = _new((nt, 32, 8), mm.FP16), _new((nt, 32, 8), mm.FP16)
        s["C"] = _new((nt, 32, 32), mm.FP32)
        s["D"] = [_new((nt, 32, 32), mm.FP32) for _ in range(3)]
        base = presets.PAPER[("cdna3", "fp16")]
        s["models"] = [mm.model_create(**base), mm.model_create(**dict(base, rd_toward_zero=True))]
        s["hists"] = [torch.empty(mm.DEVIATION_HIST_BYTES, dtype=torch.uint8, device="cuda") for _ in range(3)]
    return s


def run(s):
    return {"check": _run_check, "scan": _run_scan, "candidates": _run_candidates, "flush": _run_flush, "gemm": _run_gemm,
            "families": _run_families, "bias": _run_bias}[s["case"]["kind"]](s)


def _run_check(s):
    nt, seed, A, B, C = s["case"]["tiles"], s["seed"], s["A"], s["B"], s["C"]
    dt = (mm.FP16, mm.FP16) + FP32_OUT
    mm.generate(A, mm.FP16, 256, 0, nt, mm.GEN_FINITE_BITS, seed=seed, operand=0)
    mm.generate(B, mm.FP16, 256, 0, nt, mm.GEN_FINITE_BITS, seed=seed, operand=1)
    mm.generate(C, mm.FP32, 256, 0, nt, mm.GEN_NORMAL, seed=seed, operand=2)
    mm.emulate_mma(s["models"][0], A, B, C, s["D0"], 16, 16, 16, nt, dt)
    mm.emulate_mma(s["models"][1], A, B, C, s["D1"], 16, 16, 16, nt, dt)
    mm.stats_reset(s["stats"])
    mm.compare(s["D0"], s["D1"], nt * 256, s["stats"])
    mm.mfma_probe(mm.MFMA_F32_16X16X16_F16, A, B, C, s["Dhw"], 16, nt)
    return dict(A=A, B=B, C=C, C_value=_as_float(C), D0=s["D0"], D1=s["D1"], Dhw=s["Dhw"], stats=s["stats"].view(torch.int64))


def _run_scan(s):
    sc = s["scan"]
    sc.chunk_step(0, s["case"]["tiles"])
    return dict(A=sc.A, B=sc.B, C=sc.C, C_value=_as_float(sc.C), Dhw=sc.Dhw, stats=sc.stats.view(torch.int64))


def _run_candidates(s):
    info, nt, seed, A, B, C = s["info"], s["case"]["tiles"], s["seed"], s["A"], s["B"], s["C"]
    m, n, k = info["m"], info["n"], info["k"]
    mm.generate(A, info["a"], m * k, 0, nt, mm.GEN_NORMAL, seed=seed, operand=0)
    mm.generate(B, info["b"], n * k, 0, nt, mm.GEN_NORMAL, seed=seed, operand=1)
    mm.generate(C, mm.FP32, m * n, 0, nt, mm.GEN_NORMAL, seed=seed, operand=2)
    mm.mfma_probe(s["instr"], A, B, C, s["Dhw"], k, nt)
    mm.emulate_compare_many(s["models"], A, B, C, s["Dhw"], None, m, n, k, nt, (info["a"], info["b"]) + FP32_OUT, s["stats"])
    return dict(A=A, B=B, C=C, C_value=_as_float(C), Dhw=s["Dhw"], stats=s["stats"].view(torch.int64))


def _run_flush(s):
    nt, A, B, C = s["case"]["tiles"], s["A"], s["B"], s["C"]
    configs.config4_generate(A, B, C, 0, nt, s["seed"])
    mm.emulate_compare_many(s["models"], A, B, C, None, None, 32, 32, 8, nt, (mm.FP16, mm.FP16) + FP32_OUT, s["stats"])
    return dict(A=A, B=B, C=C, stats=s["stats"].view(torch.int64))


def _run_gemm(s):
    m, n, k = (s["case"][x] for x in "mnk")
    for h, D in zip(s["models"], s["D"]):
        mm.emulate_mma(h, s["A"], s["B"], s["C"], D, m, n, k, 1, s["dt"])
    out = dict(D=s["D"], D_value=[_as_float(D) for D in s["D"]])
    if len(s["models"]) > 1:
        mm.stats_reset(s["stats"])
        mm.compare(s["D"][0], s["D"][1], m * n, s["stats"])
        out["stats"] = s["stats"].view(torch.int64)
    if s["case"]["type"] == "fp8":
        mm.err_stats_reset(s["err"])
        mm.exact_dot_sample(s["A"], s["B"], s["D"][0], m, n, k, s["dt"], 100, s["err"])
        out.update(err_counts=s["err"].view(torch.int64)[:39], err_sums=s["err"].view(torch.float64)[39:])
    return out


def _run_families(s):
    info, nt, seed, A, B, C, D, Dhw = s["info"], s["case"]["tiles"], s["seed"], s["A"], s["B"], s["C"], s["D"], s["Dhw"]
    m, n, k, ta, tb = (info[x] for x in ("m", "n", "k", "a", "b"))
    dt = (ta, tb) + FP32_OUT
    for i, (_, ga, gb, gc) in enumerate(s["fams"]):
        mm.generate(A, ta, m * k, 0, nt, seed=seed, operand=0, **ga)
        mm.generate(B, tb, n * k, 0, nt, seed=seed, operand=1, **gb)
        mm.generate(C, mm.FP32, m * n, 0, nt, seed=seed, operand=2, **gc)
        if s["scaled"]:
            mm.generate(s["SA"], mm.E8M0, m * (k // 32), 0, nt, family=mm.GEN_UNIFORM_EXP, seed=seed, operand=3, exp_lo=120, exp_hi=134)
            mm.generate(s["SB"], mm.E8M0, n * (k // 32), 0, nt, family=mm.GEN_UNIFORM_EXP, seed=seed, operand=4, exp_lo=120, exp_hi=134)
            mm.mfma_probe_scaled(s["instr"], A, B, C, Dhw, s["SA"], s["SB"], k, nt)
            mm.emulate_mma_scaled(s["model"], A, B, C, D, s["SA"], s["SB"], 32, m, n, k, nt, dt)
        else:
            mm.mfma_probe(s["instr"], A, B, C, Dhw, k, nt)
            mm.emulate_mma(s["model"], A, B, C, D, m, n, k, nt, dt)
        mm.compare(D, Dhw, nt * m * n, s["stats"][i * mm.STATS_BYTES:])
    return dict(A=A, B=B, C=C, D=D, Dhw=Dhw, stats=s["stats"].view(torch.int64))


def _run_bias(s):
    nt, stride, A, B, C = s["case"]["tiles"], s["case"]["stride"], s["A"], s["B"], s["C"]
    dt = (mm.FP16, mm.FP16) + FP32_OUT
    configs.bias_experiment_generate(A, B, C, 0, nt, s["seed"])
    for h, D in zip(s["models"], s["D"]):
        mm.emulate_mma(h, A, B, C, D, 32, 32, 8, nt, dt)
    mm.mfma_probe(mm.MFMA_F32_32X32X8_F16, A, B, C, s["D"][2], 8, nt)
    for D, h in zip(s["D"], s["hists"]):
        mm.deviation_hist_reset(h)
        mm.deviation_sample(A, B, C, D, 32, 32, 8, nt, dt, stride, configs.BIAS_BIN_EXP, h)
    return dict(A=A, B=B, C=C, C_value=_as_float(C), D=s["D"], D_value=[_as_float(D) for D in s["D"]],
                counts=[h.view(torch.int64)[:69] for h in s["hists"]], sums=[h.view(torch.float64)[69:] for h in s["hists"]])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    """Bytes: operands written by the generators or read, accumulators, outputs; flops: two per product of every model
    and of the native instruction."""
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        e = {"fp8": 1, "bf16": 2, "fp16": 2}.get(case["type"], 4)
        models = len(_gemm_models(case["type"]))
        return dict(bytes=(m + n) * k * e + 4 * m * n * (1 + models), flops=2 * models * m * n * k)
    if kind == "families":
        instr = INSTRUCTIONS[case["instr"]]
        info = mm.mfma_info(instr)
        m, n, k, nf, models, outs = info["m"], info["n"], info["k"], len(_families(instr)), 2, 2
        e = mm.ELEM_BYTES[info["a"]]
    else:
        m, n, k, e, nf, models, outs = {"check": (16, 16, 16, 2, 1, 3, 3),
                                        "scan": (16, 16, 16, 2 if case.get("type") == "bf16" else 1, 1, 17, 1),
                                        "flush": (32, 32, 8, 2, 1, 3, 0), "bias": (32, 32, 8, 2, 1, 3, 3),
                                        "candidates": tuple(int(x) for x in case.get("shape", "0x0x0").split("x")) + (2, 1, 17, 1)}[kind]
    nt = case["tiles"]
    return dict(bytes=nf * nt * ((m + n) * k * e + 4 * m * n * (1 + outs)), flops=nf * nt * 2 * m * n * k * models)


def tolerance(case):
    # Bit patterns and counts are whole numbers and stay the same.  The binary64 sums of the error statistics and of the
    # deviation histogram are added up in no fixed order (up to 1.7e7 values: two passes differ by 2e-15 of the result,
    # another tree of partial sums by a few thousand roundings at most).
    if case["kind"] == "bias" or (case["kind"] == "gemm" and case["type"] == "fp8"):
        return {"rel": 1e-11, "max": 1e-10}
    return "exact"


# ---- the same values from plain 64-bit arithmetic -------------------------------------------------------------------

def _philox(seed, operand, blocks):
    """Philox4x32-10 (Salmon et al., SC'11): four 32-bit words for each 64-bit counter, as int64."""
    mask = 0xFFFFFFFF

    def mul(x, c):                                              # the two halves of a 32 x 32-bit product
        lo, hi = x * (c & 0xFFFF), x * (c >> 16)
        mid = (lo >> 16) + hi
        return (mid >> 16) & mask, ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)

    c0, c1 = blocks & mask, (blocks >> 32) & mask
    c2, c3 = torch.full_like(c0, operand), torch.zeros_like(c0)
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        h0, l0 = mul(c0, 0xD2511F53)
        h1, l1 = mul(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return torch.stack((c0, c1, c2, c3), dim=-1)


def _normals(seed, operand, shape):
    """The N(0,1) stream in binary64: Box-Muller on pairs of words."""
    n = math.prod(shape)
    w = _philox(seed, operand, torch.arange((n + 3) // 4, device="cuda")).reshape(-1, 2).double()
    radius = torch.sqrt(-2.0 * torch.log((w[:, 0] + 0.5) * 2.0 ** -32))
    # (the angle: the word's top two bits name the quarter turn, the centre of the cell of the other thirty the place in it)
    phi = (w[:, 1] + 0.5) * (2.0 ** -32 * 2.0 * math.pi)
    return torch.stack((radius * torch.cos(phi), radius * torch.sin(phi)), dim=-1).reshape(-1)[:n].reshape(shape)


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        a, b, c, _, _ = _gemm_operands(case, seed)
        d = a.double() @ b.double().t() + c.double()
        return dict(D_value=[d] * len(_gemm_models(case["type"])))
    if kind in ("check", "scan"):
        return dict(C_value=_normals(seed, 2, (case["tiles"], 16, 16)))
    if kind == "candidates":
        m, n, _ = (int(x) for x in case["shape"].split("x"))
        return dict(C_value=_normals(seed, 2, (case["tiles"], m, n)))
    if kind == "bias":
        nt = case["tiles"]
        a, b = ((1000.0 * _normals(seed, o, (nt, 32, 8))).float().half().double() for o in (0, 1))
        c = _normals(seed, 2, (nt, 32, 32))
        d = torch.matmul(a, b.transpose(1, 2).contiguous()) + c.float().double()
        return dict(C_value=c, D_value=[d] * 3)
    return None                                                 # counts and bit patterns: no value that 64 bits approach

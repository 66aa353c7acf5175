// GTR-FDPA on FP8 operands, groups of sixteen in two halves, with a narrow sum inside a half (F of 10 to 17): products and aligned terms
// in packed binary16, as the packed T-FDPA kernel has them, and the ends of TR-FDPA in binary64.
//
// A wavefront owns 16 x 16 outputs (R = 4: four rows of one column per lane) or half the rows of such a block (R = 2) and needs nobody
// else: it stages 32 k of its sixteen rows of A and of B by itself, eight elements per lane and operand.
//   * The maximum exponents of the four halves in 32 k come from the matrix cores.  An element is represented by 16^(e' + const), e' its
//     unnormalised exponent from the smallest upward, a zero (where zero terms stay out of the maxima) by 0: the sum of eight products of
//     such numbers lies in [16^x, 8 16^x], so x is the result's exponent field divided by 4, and 0 where no term takes part.  The codes go
//     from the lanes that loaded them straight into v_mfma_f32_16x16x32_bf16, whose lane group g holds the half g: the other groups'
//     codes of A are zero.
//   * Rows are scaled by one power of two per operand and 32 k, so that the largest product lies below 2^15: v_pk_mul_f16 forms two
//     products exactly where a half's maximum lies at most 37 - F places below the largest elements' product, and a second one by
//     2^(F - e_max - 24), rounding toward zero, cuts them at binary16's smallest subnormal, the sum's unit.  Eight terms are added up by
//     v_mfma_f32_16x16x32_f16 against zeros and ones, in the lane that owns the output.
//   * The two sums are merged as integers: what the larger maximum's half lies above the other is an arithmetic shift, which rounds down.
// Groups below that window, and 32 k that hold a NaN or an infinity, are formed term by term in binary32 by their lanes.
//
// Measured (MI355X, gfx950's FP8 set), the tiled kernels, which spend four instructions on a term where this one spends one, and this
// one: 2^13 tiles of 16x16x32, E4M3 x E5M2, N(0,1) 29 -> 17 us, all finite patterns (groups below the window in most wavefronts)
// 27 -> 23, all patterns 40 -> 25; block-scaled, 2^11 tiles of 16x16x128 37 -> 17 us; 1024^3 308 -> 197.  Bound: the vector ALU, busy 0.77 of
// the time; 17.5 instructions per term and output before, 11.5 now, most of them in the groups' ends.
#include "emulate_tiled.hpp"

namespace mmaemu {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

struct PackedRdArgs {
    int32_t F, Fm, F2, Fc, drop;
    uint32_t flags, nan_bits;
    int32_t ebase;               // Exp of a product = e'_a + e'_b + ebase
    int32_t t_a, t_b;            // exponents that the rows' largest elements are scaled to
    const uint8_t *sa, *sb;      // E8M0 scale codes, one per 32 k, or null
};

constexpr int PRD_STRIDE = 32 + 8;          // halves per staged row; 80 bytes: sixteen rows' 128-bit words lie on different banks

template <int T> __device__ __forceinline__ half2v fp8_pair(uint32_t raw, float scale, bool high)
{
    if constexpr (T == MMAEMU_FP8_E4M3) return high ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(raw, scale, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(raw, scale, false);
    else return high ? __builtin_amdgcn_cvt_scalef32_pk_f16_bf8(raw, scale, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_bf8(raw, scale, false);
}
__device__ __forceinline__ half2v word_half2(uint32_t x) { return __builtin_bit_cast(half2v, x); }

// largest of eight elements' magnitude codes
__device__ __forceinline__ uint32_t largest_code(uint2 raw)
{
    const uint32_t a = pk_max_u16(raw.x & 0x007F007Fu, (raw.x >> 8) & 0x007F007Fu), b = pk_max_u16(raw.y & 0x007F007Fu, (raw.y >> 8) & 0x007F007Fu);
    const uint32_t m = pk_max_u16(a, b), lo = m & 0xFFFFu, hi = m >> 16;
    return lo > hi ? lo : hi;
}

// codes 2^(4 e' + one - 127) of eight elements, bfloat16; `zero`: 0x00010001 where zeros count like the smallest exponent
template <int T> __device__ __forceinline__ uint4 exponent_codes(uint2 raw, uint32_t one, uint32_t zero, bool special)
{
    const uint32_t h[4] = {__builtin_amdgcn_perm(raw.x, raw.x, 0x010C000Cu), __builtin_amdgcn_perm(raw.x, raw.x, 0x030C020Cu),
                           __builtin_amdgcn_perm(raw.y, raw.y, 0x010C000Cu), __builtin_amdgcn_perm(raw.y, raw.y, 0x030C020Cu)};     // byte << 8
    const uint32_t base = ((one - 4u) << 7) * 0x10001u;
    uint32_t x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t e = T == MMAEMU_FP8_E5M2 ? (h[q] >> 1) & 0x3E003E00u : (h[q] >> 2) & 0x1E001E00u;                  // 4 E at the exponent field
        e = pk_add_u16(pk_max_u16(e, 0x02000200u), base);
        typedef unsigned short u16x2_ __attribute__((ext_vector_type(2)));
        const u16x2_ one2 = {1, 1};
        const u16x2_ live = __builtin_elementwise_min(__builtin_bit_cast(u16x2_, (h[q] & 0x7F007F00u) | zero), one2);
        x[q] = __builtin_bit_cast(uint32_t, (u16x2_)(__builtin_bit_cast(u16x2_, e) * live));
    }
    if (__builtin_expect(special, 0)) {                       // NaN and infinities stay out of the maxima (their groups are settled apart)
        constexpr uint32_t SPECIAL = T == MMAEMU_FP8_E5M2 ? 0x7C00u : 0x7F00u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((h[q] & 0x7F00u) >= SPECIAL) x[q] &= 0xFFFF0000u;
            if (((h[q] >> 16) & 0x7F00u) >= SPECIAL) x[q] &= 0x0000FFFFu;
        }
    }
    return make_uint4(x[0], x[1], x[2], x[3]);
}

template <int TA, int TB, int R, bool SC>
__global__ void __launch_bounds__(256)
emulate_packed_rd_kernel(PackedRdArgs pa, const uint8_t *__restrict__ A, const uint8_t *__restrict__ B, const uint32_t *Cm, uint32_t *D,
                         uint32_t m, uint32_t n, uint32_t k, uint64_t nitems, uint32_t bm_count, uint32_t bn_count, uint32_t xcd_remap)
{
    constexpr int WAVES = 4, PARTS = 4 / R, STRIDE = PRD_STRIDE;
    __shared__ __attribute__((aligned(16))) uint16_t lds[WAVES][2][16 * STRIDE];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t g4 = lane >> 4, c16 = lane & 15u;
    uint16_t *const va = lds[wave][0], *const vb = lds[wave][1];

    const uint32_t wg = xcd_remap ? (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const uint64_t unit = (uint64_t)wg * WAVES + wave, item = unit / PARTS;
    if (item >= nitems) return;                               // (no barriers below: wavefronts are on their own)
    const uint32_t part = (uint32_t)(unit % PARTS);
    uint64_t tile; uint32_t rem;
    split_item(item, bm_count * bn_count, tile, rem);
    const uint32_t i0 = (rem / bn_count) * 16, j0 = (rem % bn_count) * 16;
    // row mm of the matrix instructions is row row_of(mm) of the block: a lane's rows 4 g4 + r, r < R, are the part's own
    auto row_of = [&](uint32_t mm) -> uint32_t { return (mm & ~3u) | ((mm + part * R) & 3u); };
    const uint64_t row_a = tile * m + i0 + row_of(c16), row_b = tile * n + j0 + c16;
    const uint8_t *const src_a = A + row_a * k + 8 * g4, *const src_b = B + row_b * k + 8 * g4;

    uint32_t d[R];
    uint64_t place[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        place[r] = (tile * m + i0 + row_of(4 * g4 + r)) * (uint64_t)n + j0 + c16;
        d[r] = Cm[place[r]];
    }
    const uint32_t nblk = k / 32;
    const uint8_t *scale_a[SC ? R : 1], *scale_b = nullptr;
    if constexpr (SC) {
#pragma unroll
        for (int r = 0; r < R; ++r) scale_a[r] = pa.sa + (tile * m + i0 + row_of(4 * g4 + r)) * (uint64_t)nblk;
        scale_b = pa.sb + row_b * nblk;
    }

    // binary16 (and binary64) arithmetic rounds toward zero from here on: the packed scaling's cut; all other such results are exact
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3" ::: "memory");
#endif
    // selectors: ones in the eight k places that lane group g4 holds of the terms, in result row 4 g4 + r
    half8v sel[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const _Float16 x = c16 == 4 * g4 + r ? (_Float16)1.0f : (_Float16)0.0f;
        sel[r] = half8v{x, x, x, x, x, x, x, x};
    }
    const uint32_t zeros_count = (pa.flags & FL_SKIP_ZERO) ? 0u : 0x00010001u;
    const float merge = __uint_as_float((uint32_t)(127 + 24 + pa.Fm - pa.F) << 23);
    const float4v zero4 = {0.0f, 0.0f, 0.0f, 0.0f};

    uint2 raw_a = *reinterpret_cast<const uint2 *>(src_a), raw_b = *reinterpret_cast<const uint2 *>(src_b);
    for (uint32_t k0 = 0; k0 < k; k0 += 32) {
        // ---- 32 k: the operands' scales, exponent codes and values ----
        uint32_t top = largest_code(raw_a) | (largest_code(raw_b) << 16);
#if defined(__HIP_DEVICE_COMPILE__)
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x111, 0xF, 0xF, false));
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x112, 0xF, 0xF, false));
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x114, 0xF, 0xF, false));
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x118, 0xF, 0xF, false));
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x142, 0xA, 0xF, false));
        top = pk_max_u16(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x143, 0xC, 0xF, false));
        top = (uint32_t)__builtin_amdgcn_readlane((int)top, 63);
#endif
        const uint32_t top_a = top & 0xFFFFu, top_b = top >> 16;
        constexpr uint32_t SPECIAL_A = TA == MMAEMU_FP8_E5M2 ? 0x7Cu : 0x7Fu, SPECIAL_B = TB == MMAEMU_FP8_E5M2 ? 0x7Cu : 0x7Fu;
        const bool special = top_a >= SPECIAL_A || top_b >= SPECIAL_B;
        const int Ea = (int)(top_a >> Fmt<TA>::MB), Eb = (int)(top_b >> Fmt<TB>::MB);
        const int down_a = pa.t_a + Fmt<TA>::BIAS - (Ea ? Ea : 1), down_b = pa.t_b + Fmt<TB>::BIAS - (Eb ? Eb : 1);       // (places that the values are moved by)
        const uint4 xa = exponent_codes<TA>(raw_a, 64u, zeros_count, special), xb = exponent_codes<TB>(raw_b, 67u, zeros_count, special);
        const float sc_a = __uint_as_float((uint32_t)(127 + down_a) << 23), sc_b = __uint_as_float((uint32_t)(127 + down_b) << 23);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        *reinterpret_cast<uint4 *>(va + c16 * STRIDE + 8 * g4) = make_uint4(
            __builtin_bit_cast(uint32_t, fp8_pair<TA>(raw_a.x, sc_a, false)), __builtin_bit_cast(uint32_t, fp8_pair<TA>(raw_a.x, sc_a, true)),
            __builtin_bit_cast(uint32_t, fp8_pair<TA>(raw_a.y, sc_a, false)), __builtin_bit_cast(uint32_t, fp8_pair<TA>(raw_a.y, sc_a, true)));
        *reinterpret_cast<uint4 *>(vb + c16 * STRIDE + 8 * g4) = make_uint4(
            __builtin_bit_cast(uint32_t, fp8_pair<TB>(raw_b.x, sc_b, false)), __builtin_bit_cast(uint32_t, fp8_pair<TB>(raw_b.x, sc_b, true)),
            __builtin_bit_cast(uint32_t, fp8_pair<TB>(raw_b.y, sc_b, false)), __builtin_bit_cast(uint32_t, fp8_pair<TB>(raw_b.y, sc_b, true)));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (k0 + 32 < k) {
            raw_a = *reinterpret_cast<const uint2 *>(src_a + k0 + 32);
            raw_b = *reinterpret_cast<const uint2 *>(src_b + k0 + 32);
        }
        int scale_exp[R];
        bool scale_nan[R];
#pragma unroll
        for (int r = 0; r < R; ++r) { scale_exp[r] = 0; scale_nan[r] = false; }
        if constexpr (SC) {
            const uint32_t y = scale_b[k0 / 32];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t x = scale_a[r][k0 / 32];
                scale_exp[r] = (int)(x + y) - 254;
                scale_nan[r] = x == 0xFFu || y == 0xFFu;
            }
        }
        // the scale of a half with maximum code x is 2^(most - x); x at `most` is the window's end
        const int most = pa.F - 24 - (down_a + down_b) + 1 - pa.ebase;
        const uint32_t window = (uint32_t)(most > 1 ? most : 1);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            uint32_t x[2][R];
            uint32_t least = 0xFFFFFFFFu;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool mine = g4 == (uint32_t)(2 * g + h);
                const uint4 xm = make_uint4(mine ? xa.x : 0u, mine ? xa.y : 0u, mine ? xa.z : 0u, mine ? xa.w : 0u);
                const float4v mx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8v, xm), __builtin_bit_cast(bf16x8v, xb), zero4, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    x[h][r] = __float_as_uint(mx[r]) >> 25;                    // 0: no term takes part
                    least = min(x[h][r] - 1u, least);
                }
            }
            int32_t T[2][R];                                                  // the halves' sums, in units of 2^(e_max - Fm)
            uint32_t dn[R];
            float ieee[R];
            if (__builtin_expect(special || __any(least < window - 1u), 0)) {
#pragma unroll
                for (int r = 0; r < R; ++r) ieee[r] = 0.0f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float scale[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        T[h][r] = 0;
                        int e = 127 + 24 + most - (int)x[h][r];               // 2^(F - e_max) in the scaled values
                        e = x[h][r] ? e : 127;
                        scale[r] = __uint_as_float((uint32_t)(e < 1 ? 1 : (e > 254 ? 254 : e)) << 23);
                    }
#pragma unroll 1
                    for (int q = 0; q < 8; ++q) {
                        const uint32_t o = 8 * (2 * g + h) + q;
                        const float b = (float)__builtin_bit_cast(_Float16, vb[c16 * STRIDE + o]);
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float p = (float)__builtin_bit_cast(_Float16, va[(4 * g4 + r) * STRIDE + o]) * b;
                            T[h][r] += (int32_t)(p * scale[r]);
                            ieee[r] += p;
                        }
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) T[h][r] = (int32_t)((uint32_t)T[h][r] << (pa.Fm - pa.F));
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t o = 8 * (2 * g + h);
                    const uint4 bw = *reinterpret_cast<const uint4 *>(vb + c16 * STRIDE + o);
                    const uint32_t b[4] = {bw.x, bw.y, bw.z, bw.w};
                    float4v S = zero4;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const uint4 aw = *reinterpret_cast<const uint4 *>(va + (4 * g4 + r) * STRIDE + o);
                        const uint32_t a[4] = {aw.x, aw.y, aw.z, aw.w};
                        const uint32_t xw = max(x[h][r], window);             // (a half without terms: any finite scale)
                        const _Float16 sc = __builtin_ldexpf16((_Float16)1.0f, most - (int)xw);
                        half2v t[4];
#pragma unroll
                        for (int w = 0; w < 4; ++w) t[w] = word_half2(a[w]) * word_half2(b[w]);
#pragma unroll
                        for (int w = 0; w < 4; ++w) t[w] = t[w] * half2v{sc, sc};
                        S = __builtin_amdgcn_mfma_f32_16x16x32_f16(sel[r], half8v{t[0][0], t[0][1], t[1][0], t[1][1], t[2][0], t[2][1], t[3][0], t[3][1]}, S, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) T[h][r] = (int32_t)(S[r] * merge);
                }
            }
            // ---- the merged sum (steps 3 to 5 of GTR-FDPA), then TR-FDPA's last steps ----
            double Td[R], v[R];
            int em[R];
            bool have[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t xm = max(x[0][r], x[1][r]);
                Td[r] = (double)((T[0][r] >> min(xm - x[0][r], 31u)) + (T[1][r] >> min(xm - x[1][r], 31u)));
                em[r] = (int)xm - 1 + pa.ebase + scale_exp[r];
                have[r] = xm != 0u;
            }
            const bool low = rd_exact_all<true>(Td, em, pa.Fm, d, pa.F2, pa.Fc, pa.drop, pa.flags, v, have);
#pragma unroll
            for (int r = 0; r < R; ++r) dn[r] = __float_as_uint((float)v[r]);
            if (low && (pa.flags & FL_ZERO_POSITIVE)) {
#pragma unroll
                for (int r = 0; r < R; ++r) dn[r] = (dn[r] & 0x7FFFFFFFu) == 0 ? 0u : dn[r];
            }
            if (__builtin_expect(special, 0)) {
                // Sec. 4.2: the IEEE sum of the group's products (finite ones below 2^20 in the scaled values) and its accumulator is a
                // NaN or an infinity exactly where the group's result is
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (!(__builtin_fabsf(ieee[r]) <= 3.4028234663852886e38f)) dn[r] = __float_as_uint(ieee[r] + ((d[r] & 0x7F800000u) == 0x7F800000u ? __uint_as_float(d[r]) : 0.0f));
                }
            }
            if constexpr (SC) {
#pragma unroll
                for (int r = 0; r < R; ++r) dn[r] = scale_nan[r] ? 0x7FC00000u : dn[r];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) d[r] = dn[r];
        }
    }
    // (a NaN travels with whatever pattern the arithmetic gives it; the model's is written once here)
#pragma unroll
    for (int r = 0; r < R; ++r) D[place[r]] = (d[r] & 0x7FFFFFFFu) > 0x7F800000u ? pa.nan_bits : d[r];
}

// ---- host side ---------------------------------------------------------------------------

// Blocks below which two wavefronts share one: each stages all of it, which costs 15 %, but with fewer than a wavefront for every SIMD the
// chain of groups counts.  One wavefront and two, us: 256, 512, 1024, 2048 blocks of k = 128 12.0, 11.3, 11.5, 16.8 and 10.1, 10.0, 12.6,
// 19.1; 2^11 and 2^13 of k = 32 9.3, 17.1 and 8.5, 20.5.  The line is that of k = 128, for every k: with one group or two to a chain it
// lies higher (somewhere between 2^11 and 2^13 blocks of k = 32), for a tenth of launches of 9 us, and was not looked for.
constexpr uint64_t PRD_SPLIT_BELOW = 768;

template <int TA, int TB, int R, bool SC>
static mmaemu_status launch_packed_rd_cfg(const PackedRdArgs &pa, const void *A, const void *B, const void *Cm, void *D, uint32_t m, uint32_t n,
                                          uint32_t k, uint64_t nitems, hipStream_t s)
{
    const uint64_t blocks = (nitems * (4 / R) + 3) / 4;
    if (blocks > (1ull << 32) / 256 - 1) { set_error("emulate_mma: too many blocks"); return MMAEMU_ERR_SHAPE; }
    const uint32_t remap = (blocks % 8 == 0 && blocks >= 64) ? 1u : 0u;
    hipLaunchKernelGGL((emulate_packed_rd_kernel<TA, TB, R, SC>), dim3((uint32_t)blocks), dim3(256), 0, s, pa, (const uint8_t *)A, (const uint8_t *)B,
                       (const uint32_t *)Cm, (uint32_t *)D, m, n, k, nitems, m / 16, n / 16, remap);
    MMAEMU_HIP(hipGetLastError());
    set_last_kernel("tiled 16x16 packed halves r%d kc=32 L=16 c_mode=%d vm=%d", R, CM_RD_HALVES, SC ? 3 : 0);
    return MMAEMU_OK;
}

bool packed_rd_takes(const ModelArgs &p, uint32_t ta, uint32_t tb, uint32_t m, uint32_t n, uint32_t k, uint64_t batch, bool scaled, uint32_t block)
{
    if (p.c_mode != MMAEMU_C_AFTER_RD || p.split != MMAEMU_SPLIT_HALVES || p.L != 16 || !(p.flags & FL_SUM_EXACT)) return false;
    if (p.flags & (FL_ACC16 | FL_RZ | FL_FTZ_OUT | FL_FTZ_IN | FL_RD_AS_RZ | FL_NAN_PROPAGATE)) return false;
    // (two E5M2 operands span 64 places together, more than binary16 can scale: the tiled kernels)
    if (ta > MMAEMU_FP8_E5M2 || tb > MMAEMU_FP8_E5M2 || (ta == MMAEMU_FP8_E5M2 && tb == MMAEMU_FP8_E5M2)) return false;
    if (m % 16 != 0 || n % 16 != 0 || k % 32 != 0) return false;
    // (under the overflow rule a scaled product may count as an infinity: the tiled kernels)
    if (scaled && (block != 32 || !(p.flags & FL_WIDE_PRODUCTS))) return false;
    if (batch * (m / 16) * (n / 16) >= 1ull << 24) return false;                        // (one launch)
    // a half's sum below 2^24 units; the merged sum a 32-bit integer
    return p.F >= 10 && p.F <= 17 && p.Fm >= p.F && p.Fm <= 25;
}

mmaemu_status launch_emulate_packed_rd(const ModelArgs &p, const void *A, const void *B, const void *Cm, void *D, uint32_t m, uint32_t n,
                                       uint32_t k, uint64_t batch, uint32_t ta, uint32_t tb, hipStream_t s, const uint8_t *SA, const uint8_t *SB)
{
    PackedRdArgs pa = {};
    pa.F = p.F; pa.Fm = p.Fm; pa.F2 = p.F2; pa.Fc = p.Fc; pa.drop = p.sum_drop_distance;
    pa.flags = p.flags;
    pa.nan_bits = p.nan_bits;
    pa.ebase = 2 - fmt_info(ta).bias - fmt_info(tb).bias;
    pa.sa = SA; pa.sb = SB;
    // Products below 2^(t_a + t_b + 2): 13 together keeps them below 2^15, and F or less the window inside one factor.  A row of E5M2 is
    // held whole from T = 8 upward, one of E4M3 from -7.
    const int top = p.F < 13 ? p.F : 13;
    if (ta == tb) { pa.t_a = top / 2; pa.t_b = top - pa.t_a; }
    else if (ta == MMAEMU_FP8_E4M3) { pa.t_b = 8; pa.t_a = top - 8; }
    else { pa.t_a = 8; pa.t_b = top - 8; }
    const uint64_t nitems = batch * (m / 16) * (n / 16);
    const bool halved = nitems < PRD_SPLIT_BELOW;
#define GO(X, Y)                                                                                                                                      \
    if (ta == X && tb == Y) {                                                                                                                         \
        if (SA) return halved ? launch_packed_rd_cfg<X, Y, 2, true>(pa, A, B, Cm, D, m, n, k, nitems, s) : launch_packed_rd_cfg<X, Y, 4, true>(pa, A, B, Cm, D, m, n, k, nitems, s); \
        return halved ? launch_packed_rd_cfg<X, Y, 2, false>(pa, A, B, Cm, D, m, n, k, nitems, s) : launch_packed_rd_cfg<X, Y, 4, false>(pa, A, B, Cm, D, m, n, k, nitems, s);        \
    }
    GO(MMAEMU_FP8_E4M3, MMAEMU_FP8_E4M3)
    GO(MMAEMU_FP8_E4M3, MMAEMU_FP8_E5M2)
    GO(MMAEMU_FP8_E5M2, MMAEMU_FP8_E4M3)
#undef GO
    set_error("emulate_mma: the packed kernel takes no two E5M2 operands");
    return MMAEMU_ERR_UNSUPPORTED;
}

} // namespace mmaemu

// T-FDPA on FP8 operands with a narrow sum (F up to 17): products and aligned terms in packed binary16.
//
// What bounds the model on the vector ALU is the work per term.  The tiled kernels take 4.5 instructions: two halves of a packed
// operation for the maximum exponent, two multiplications, a conversion and the sum.  FP8 operands with F <= 17 allow one and a
// matrix instruction:
//   * a product of two FP8 values has at most 8 significant bits, so binary16 holds it exactly: v_pk_mul_f16, two products;
//   * a second packed multiplication by 2^(F - e_max - 24), under the rounding mode "toward zero", puts the sum's unit at binary16's
//     smallest subnormal, 2^-24: terms that reach above it keep their 8 bits, what lies below it is cut -- RZ_F itself;
//   * v_mfma_f32_16x16x32_f16 against a matrix of zeros and ones adds up eight such terms of each of 64 outputs, exactly (all are
//     multiples of the unit, and (L + 1) 2^(F+2) <= 2^24); the ones choose the result column, so that the four outputs of a lane
//     fill one accumulator and come out transposed: four neighbours of a row of D in each lane.  (v_dot2_f32_f16 with ones does the
//     same without the transposition at two instructions per eight terms: a 4096^3 pass with its exact dots took 4960 us, against 4270
//     for the first kernel with the matrix sum.)
//   * the maximum exponent comes from the matrix cores too.  An element is represented by 2^(8 (Exp - Exp_row)), Exp_row the largest
//     exponent of its row in the group; the dot product of two such rows lies in [2^(8 x), 32 * 2^(8 x)) with x the
//     group's maximum relative to the two rows', so x is the result's exponent field divided by 8: one shift.
// Rows are scaled by 2^(T - Exp_row), group by group, when they are converted, so that data of any size uses binary16's range.  The
// matrix result and the scale hold maxima down to x = -15, and none lies lower: one of the operands is E4M3, whose exponents
// (zeros and subnormals included) span 14 places, so the product at the other row's largest element has x >= -14.  The accumulator may
// lie up to 9 places above the rows' product; a wavefront whose accumulators lie further up, or that holds a NaN or an infinity,
// scales in two steps.
//
// Measured (MI355X), F = 14, N(0,1) data, the tiled kernel and this one: groups of 32, E4M3 x E5M2, 4096^3 9.13 -> 4.03 ms (17.0 T
// terms/s; 2.1 vector instructions per term at 0.9 of the nominal rate, most of them of the packed kind that issues at 0.95 of it),
// 2048^3 1.21 -> 0.53 ms, 1024^3 172 -> 91 us, 100 x 77 x 320 27 -> 15.5 us; all bit patterns (a NaN or an infinity in every
// wavefront) 2048^3 2.21 -> 1.06 ms, accumulators of 10^6 1.21 -> 1.03 ms.  Groups of 16, E4M3 x E4M3, 4096^3 9.96 -> 5.25 ms;
// 2048^3 with one large element per row and 32 k 1.32 -> 1.29 ms (4.52 while a row had one scale for both its groups and groups far
// below it went to a routine of their own; without that routine the kernels need no scratch memory: groups of 32 4.17 -> 4.03 ms,
// groups of 16 6.43 -> 5.25).
// 64 x 64 blocks of eight wavefronts hold two blocks of 16 columns each: with four (and half the wavefronts) the loop was 8 % faster,
// but its second form, which the last two of these take, sent 160 registers to scratch memory and ran at half the tiled kernel's speed.
#include "emulate_tiled.hpp"

namespace mmaemu {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef _Float16 half4v __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

struct PackedArgs {
    int32_t F;
    uint32_t flags, out_mask, nan_bits;
    int32_t top;                 // T_A + T_B: the products' largest exponent in the scaled rows
    int32_t t_a, t_b;            // T of A's and of B's rows
    uint32_t reach23;            // largest e_max less the rows' exponents, plus 16, that one factor scales, at the exponent field
    int32_t c2;                  // (127 + 127 + F - top - 24) at the exponent field: what the rows' exponents less e_max make the scale with
};

constexpr int PACKED_STRIDE = 32 + 8;       // halves per staged row; 80 bytes: sixteen rows' 128-bit words lie on different banks
constexpr int PACKED_ROOM = 9;             // places that the accumulator's exponent may lie above the rows' product

template <int T> struct Fp8 {
    static constexpr int MB = Fmt<T>::MB, BIAS = Fmt<T>::BIAS;
    static constexpr uint32_t SPECIAL = T == MMAEMU_FP8_E5M2 ? 0x7Cu : 0x7Fu;        // magnitudes from here on: infinity or NaN
    static __device__ __forceinline__ half2v pair(uint32_t raw, float scale, bool high)
    {
        if constexpr (T == MMAEMU_FP8_E4M3) return high ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(raw, scale, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(raw, scale, false);
        else return high ? __builtin_amdgcn_cvt_scalef32_pk_f16_bf8(raw, scale, true) : __builtin_amdgcn_cvt_scalef32_pk_f16_bf8(raw, scale, false);
    }
};

__device__ __forceinline__ uint32_t as_u32(half2v x) { uint32_t r; __builtin_memcpy(&r, &x, 4); return r; }
__device__ __forceinline__ half2v as_half2(uint32_t x) { half2v r; __builtin_memcpy(&r, &x, 4); return r; }

// The largest exponents of the wavefront's groups, relative to the rows' (result layout: row c16, columns 4 g4 + v of each block).
template <int NC, int L>
__device__ __forceinline__ void packed_maxima(const uint16_t *xa, const uint16_t *xb, uint32_t g4, uint32_t c16, float4v (&mx)[NC])
{
    constexpr int STRIDE = PACKED_STRIDE;
    const float4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (L == 32) {
        const bf16x8v fa = *reinterpret_cast<const bf16x8v *>(xa + c16 * STRIDE + 8 * g4);
#pragma unroll
        for (int c = 0; c < NC; ++c) mx[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8v *>(xb + (16 * c + c16) * STRIDE + 8 * g4), fa, zero, 0, 0, 0);
    } else {
        const short4v fa = *reinterpret_cast<const short4v *>(xa + c16 * STRIDE + 4 * g4);
#pragma unroll
        for (int c = 0; c < NC; ++c) mx[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const short4v *>(xb + (16 * c + c16) * STRIDE + 4 * g4), fa, zero, 0, 0, 0);
    }
}

// rho of an exact sum V in units of 2^(em - F), an integer below 2^24: the product is exact and normal (or zero)
__device__ __forceinline__ uint32_t packed_finish(const PackedArgs &pa, float V, uint32_t em)
{
    uint32_t o = __float_as_uint(V * __uint_as_float(em - ((uint32_t)pa.F << 23)));
    if (pa.flags & FL_RZ) o &= pa.out_mask;              // (nothing to round; RZ-E8M13 cuts further)
    return o;
}

// A workgroup of WR * WC wavefronts owns WR * 16 rows and WC * NC * 16 columns of one tile's D; a wavefront 16 rows and NC blocks of
// 16 columns.  A lane multiplies four rows with one column of each block, and owns four neighbouring outputs of one row of each.
// KC = 32 k are staged at a time.
template <int TA, int TB, int WR, int WC, int NC, int L>
__global__ void __launch_bounds__(64 * WR * WC) __attribute__((amdgpu_waves_per_eu(4, 4)))
emulate_packed_kernel(PackedArgs pa, const uint8_t *__restrict__ A, const uint8_t *__restrict__ B, const uint32_t *Cm, uint32_t *D,
                      uint32_t m, uint32_t n, uint32_t k, uint32_t bm_count, uint32_t bn_count, uint32_t xcd_remap)
{
    constexpr int KC = 32, ROWS_A = 16 * WR, ROWS_B = 16 * WC * NC, THREADS = 64 * WR * WC;
    constexpr int STRIDE = PACKED_STRIDE;
    constexpr int R = 4;
    __shared__ __attribute__((aligned(16))) uint16_t va[ROWS_A * STRIDE], vb[ROWS_B * STRIDE];      // scaled values, binary16
    __shared__ __attribute__((aligned(16))) uint16_t xa[ROWS_A * STRIDE], xb[ROWS_B * STRIDE];      // 2^(8 (Exp - Exp_row)), bfloat16
    __shared__ __attribute__((aligned(16))) int32_t ea[KC / L][ROWS_A];          // Exp_row 2^23 of every group
    __shared__ __attribute__((aligned(16))) int32_t eb[KC / L][ROWS_B];

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t wr = wave % WR, wc = wave / WR;
    const uint32_t g4 = lane >> 4, c16 = lane & 15u;

    const uint32_t wg = xcd_remap ? (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    uint64_t tile; uint32_t rem;
    split_item(wg, bm_count * bn_count, tile, rem);
    const uint32_t i0 = (rem / bn_count) * ROWS_A, j0 = (rem % bn_count) * ROWS_B;

    // staging: eight consecutive k of one row per thread and step, four threads to a row
    constexpr int SA_ = (ROWS_A * 4 + THREADS - 1) / THREADS, SB_ = (ROWS_B * 4 + THREADS - 1) / THREADS;
    static_assert(ROWS_A * 4 % 64 == 0 && ROWS_B * 4 % 64 == 0, "whole wavefronts stage");
    uint2 raw_a[SA_], raw_b[SB_];
    auto row_a = [&](uint32_t r) -> const uint8_t * { const uint32_t i = i0 + r; return A + (tile * m + (i < m ? i : m - 1)) * (uint64_t)k; };
    auto row_b = [&](uint32_t r) -> const uint8_t * { const uint32_t j = j0 + r; return B + (tile * n + (j < n ? j : n - 1)) * (uint64_t)k; };
    const uint8_t *src_a[SA_], *src_b[SB_];
#pragma unroll
    for (int i = 0; i < SA_; ++i) { const uint32_t u = tid + THREADS * i; src_a[i] = row_a((u / 4) % ROWS_A) + 8 * (u % 4); }
#pragma unroll
    for (int i = 0; i < SB_; ++i) { const uint32_t u = tid + THREADS * i; src_b[i] = row_b((u / 4) % ROWS_B) + 8 * (u % 4); }
    auto prefetch = [&](uint32_t k0) {
#pragma unroll
        for (int i = 0; i < SA_; ++i) raw_a[i] = *reinterpret_cast<const uint2 *>(src_a[i] + k0);
#pragma unroll
        for (int i = 0; i < SB_; ++i) raw_b[i] = *reinterpret_cast<const uint2 *>(src_b[i] + k0);
    };
    const uint32_t ftz_in = pa.flags & FL_FTZ_IN;
    auto stage = [&](auto type_c, const uint2 raw, uint32_t row, uint32_t part, uint16_t *lv, uint16_t *lx, auto &le, int t_shift, uint32_t one) {
        constexpr int T = decltype(type_c)::value;
        using P = Fp8<T>;
        // the largest magnitude code of the row in the group, L / 8 threads (codes order like exponents)
        const uint32_t mx0 = raw.x & 0x007F007Fu, mx1 = (raw.x >> 8) & 0x007F007Fu, mx2 = raw.y & 0x007F007Fu, mx3 = (raw.y >> 8) & 0x007F007Fu;
        uint32_t mx = pk_max_u16(pk_max_u16(mx0, mx1), pk_max_u16(mx2, mx3));
        mx = pk_max_u16(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0xB1, 0xF, 0xF, true));      // lanes 1, 0, 3, 2 of the quad
        if constexpr (L == 32) mx = pk_max_u16(mx, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, 0x4E, 0xF, 0xF, true));      // lanes 2, 3, 0, 1
        const uint32_t lo = mx & 0xFFFFu, hi = mx >> 16, top = lo > hi ? lo : hi;
        const uint32_t E = top >> P::MB ? top >> P::MB : 1u;                                                // Exp_row + bias
        // exponent codes: max(E, 1) at bit 10 of every half, relative to the row's
        uint32_t h[4] = {__builtin_amdgcn_perm(raw.x, raw.x, 0x010C000Cu), __builtin_amdgcn_perm(raw.x, raw.x, 0x030C020Cu),
                         __builtin_amdgcn_perm(raw.y, raw.y, 0x010C000Cu), __builtin_amdgcn_perm(raw.y, raw.y, 0x030C020Cu)};     // byte << 8
        const uint32_t base = (one << 7) - (E << 10), base2 = (base & 0xFFFFu) * 0x10001u;
        uint32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t e10 = T == MMAEMU_FP8_E5M2 ? h[q] & 0x7C007C00u : (h[q] >> 1) & 0x3C003C00u;
            e10 = pk_max_u16(e10, 0x04000400u);
            x[q] = pk_add_u16(e10, base2);
            if constexpr (T == MMAEMU_FP8_E5M2) {
                // (more than 15 places below the row's largest: zero)
                typedef short i16x2 __attribute__((ext_vector_type(2)));
                i16x2 s, z = {0, 0};
                __builtin_memcpy(&s, &x[q], 4);
                s = __builtin_elementwise_max(s, z);
                __builtin_memcpy(&x[q], &s, 4);
            }
        }
        if (__builtin_expect(__any(top >= P::SPECIAL), 0)) {
            // NaN and infinities: a NaN for a code, so that every group's maximum that meets one is a NaN
            auto mark = [&](uint32_t w, uint32_t &x0, uint32_t &x1) {
                if ((w & 0x7Fu) >= P::SPECIAL) x0 = (x0 & 0xFFFF0000u) | 0x7FC0u;
                if (((w >> 8) & 0x7Fu) >= P::SPECIAL) x0 = (x0 & 0xFFFFu) | 0x7FC00000u;
                if (((w >> 16) & 0x7Fu) >= P::SPECIAL) x1 = (x1 & 0xFFFF0000u) | 0x7FC0u;
                if (((w >> 24) & 0x7Fu) >= P::SPECIAL) x1 = (x1 & 0xFFFFu) | 0x7FC00000u;
            };
            mark(raw.x, x[0], x[1]);
            mark(raw.y, x[2], x[3]);
        }
        // values, scaled by a power of two
        uint2 r = raw;
        if (__builtin_expect(ftz_in != 0, 0)) {           // subnormals become +0
            auto flush = [&](uint32_t w) -> uint32_t {
#pragma unroll
                for (int q = 0; q < 4; ++q) if (((w >> (8 * q)) & 0x7Fu) < (1u << P::MB)) w &= ~(0xFFu << (8 * q));
                return w;
            };
            r.x = flush(r.x); r.y = flush(r.y);
#if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("" : "+v"(r.x), "+v"(r.y));      // (a branch, not forty selects on the way)
#endif
        }
        const float sc = __uint_as_float((uint32_t)(127 + t_shift + P::BIAS - (int)E) << 23);
        uint4 v;
        v.x = as_u32(P::pair(r.x, sc, false)); v.y = as_u32(P::pair(r.x, sc, true));
        v.z = as_u32(P::pair(r.y, sc, false)); v.w = as_u32(P::pair(r.y, sc, true));
        *reinterpret_cast<uint4 *>(lv + row * STRIDE + 8 * part) = v;
        *reinterpret_cast<uint4 *>(lx + row * STRIDE + 8 * part) = make_uint4(x[0], x[1], x[2], x[3]);
        if (part % (L / 8) == 0) le[part / (L / 8)][row] = ((int)E - P::BIAS) * (1 << 23);
    };

    // outputs: row c16 of the wavefront's sixteen, columns 4 g4 .. 4 g4 + 3 of each block
    uint32_t d[NC][4];
    const uint32_t oi = i0 + 16 * wr + c16;
    const uint64_t orow = (tile * m + (oi < m ? oi : m - 1)) * (uint64_t)n;
    auto out_col = [&](int c) -> uint32_t { return j0 + (wc * NC + c) * 16 + 4 * g4; };
    const bool wide = (n & 3u) == 0 && ((reinterpret_cast<uintptr_t>(Cm) | reinterpret_cast<uintptr_t>(D)) & 15) == 0;       // (uniform)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t j = out_col(c);
        if (wide) {
            const uint4 v = *reinterpret_cast<const uint4 *>(Cm + orow + (j < n ? j : n - 4));
            d[c][0] = v.x; d[c][1] = v.y; d[c][2] = v.z; d[c][3] = v.w;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) d[c][v] = Cm[orow + (j + v < n ? j + v : n - 1)];
        }
    }

    const uint32_t C1 = (uint32_t)(pa.F + 254) << 23;
    // binary16 arithmetic rounds toward zero from here on (the packed scaling's cut; its other results are exact)
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3" ::: "memory");
#endif
    // selectors: ones in the eight k places that lane group g4 holds of A, in result column 4 g4 + r
    half8v sel[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const _Float16 x = c16 == 4 * g4 + r ? (_Float16)1.0f : (_Float16)0.0f;
        sel[r] = half8v{x, x, x, x, x, x, x, x};
    }
    short4v unit;                                         // the 16 x 16 identity in bfloat16: k = 4 g4 + v, column c16
#pragma unroll
    for (int v = 0; v < 4; ++v) unit[v] = c16 == 4 * g4 + v ? (short)0x3F80 : (short)0;
    prefetch(0);
    for (uint32_t k0 = 0; k0 < k; k0 += KC) {
        if (k0) __syncthreads();
#pragma unroll
        for (int i = 0; i < SA_; ++i) {
            const uint32_t u = tid + THREADS * i;
            if (ROWS_A * 4 % THREADS == 0 || u < ROWS_A * 4) stage(std::integral_constant<int, TA>{}, raw_a[i], u / 4, u % 4, va, xa, ea, pa.t_a, 128u);
        }
#pragma unroll
        for (int i = 0; i < SB_; ++i) {
            const uint32_t u = tid + THREADS * i;
            if (ROWS_B * 4 % THREADS == 0 || u < ROWS_B * 4) stage(std::integral_constant<int, TB>{}, raw_b[i], u / 4, u % 4, vb, xb, eb, pa.t_b, 127u);
        }
        __syncthreads();
        if (k0 + KC < k) prefetch(k0 + KC);
#pragma unroll 1
        for (int g = 0; g < KC / L; ++g) {
            // ---- maximum exponents ----
            float4v mx[NC];
            const uint16_t *const xa_w = xa + 16 * wr * STRIDE + g * L, *const xb_w = xb + wc * NC * 16 * STRIDE + g * L;
            packed_maxima<NC, L>(xa_w, xb_w, g4, c16, mx);
            // (result layout: this lane's outputs)
            const int ka_o = ea[g][16 * wr + c16] + (111 << 23);
            uint32_t em[NC][4], most = 0, reach = 0;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int4 kb = *reinterpret_cast<const int4 *>(eb[g] + (wc * NC + c) * 16 + 4 * g4);
                const int kv[4] = {kb.x, kb.y, kb.z, kb.w};
#pragma unroll
                for (int v = 0; v < 4; v += 2) {
                    uint32_t w[2], x[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        w[h] = __float_as_uint(mx[c][v + h]);
                        const uint32_t kab = (uint32_t)(ka_o + kv[v + h]), ep = ((w[h] >> 3) & 0x1F800000u) + kab, ec = d[c][v + h] & 0x7F800000u;
                        em[c][v + h] = ep > ec ? ep : ec;
                        x[h] = em[c][v + h] - kab;
                    }
                    most = max(max(w[0], w[1]), most);               // (three operands in one instruction)
                    reach = max(max(x[0], x[1]), reach);
                }
            }
            // slow: some accumulator lies more places above its rows' product than one power of two of binary16 can scale by (the
            // scale is then applied in two factors), or the group is a special one (a NaN or an infinity; of an accumulator, whose
            // exponent, 255, is at least 90 above any product's)
            const bool slow = __any(most >= (17u << 26) || reach > pa.reach23) != 0;
            const float4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
            if (__builtin_expect(slow, 0)) {               // (finite powers of two, whatever the accumulators are)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) em[c][v] = min(em[c][v], 254u << 23);
            }
            // the accumulator aligned and cut like a term, in units of 2^24: the sums start from it
            float4v S[NC];
            uint32_t sc[R][NC];
            const int4 ka = *reinterpret_cast<const int4 *>(ea[g] + 16 * wr + 4 * g4);
            const int kr[R] = {ka.x, ka.y, ka.z, ka.w};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
#pragma unroll
                for (int v = 0; v < 4; ++v) S[c][v] = __builtin_truncf(__uint_as_float(d[c][v]) * __uint_as_float(C1 - em[c][v])) * 0x1p-24f;
                // the maxima once more in the layout of the products (rows 4 g4 + r, column c16): the matrix 2^(e_max) times the identity
                const uint2 packed = make_uint2(__builtin_amdgcn_perm(em[c][1], em[c][0], 0x07060302u), __builtin_amdgcn_perm(em[c][3], em[c][2], 0x07060302u));
                const float4v t = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, packed), unit, zero, 0, 0, 0);
                const uint32_t kb = (uint32_t)eb[g][(wc * NC + c) * 16 + c16] + (uint32_t)pa.c2;
                if (__builtin_expect(slow, 0)) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        // (the exponent difference as an integer: it may lie below binary32's range)
                        const int e = (int)((uint32_t)kr[r] + (uint32_t)kb - __float_as_uint(t[r])) >> 23, down = e - (127 - 24);
                        const float over = __uint_as_float((uint32_t)(127 - 24 + (down > 0 ? down : 0)) << 23);
                        const float under = __uint_as_float((uint32_t)(127 + (down < -30 ? -30 : (down > 0 ? 0 : down))) << 23);
                        sc[r][c] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(over, under));
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float s32 = __uint_as_float((uint32_t)kr[r] + (uint32_t)kb - __float_as_uint(t[r]));
                        sc[r][c] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(s32, s32));
                    }
                }
            }
            if (__builtin_expect(slow, 0)) {
                // Sec. 4.2 through the IEEE sum of the group's products and its accumulator, which is a NaN or an infinity exactly
                // where the group's result is (the scaled finite products stay below 2^16); the matrix cores form the products' part.
                // Such a sum starts from its result and keeps it through the terms.
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    float4v t;
                    if constexpr (L == 32)
                        t = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const half8v *>(vb + ((wc * NC + c) * 16 + c16) * STRIDE + 8 * g4),
                                                                   *reinterpret_cast<const half8v *>(va + (16 * wr + c16) * STRIDE + 8 * g4), zero, 0, 0, 0);
                    else
                        t = __builtin_amdgcn_mfma_f32_16x16x16f16(*reinterpret_cast<const half4v *>(vb + ((wc * NC + c) * 16 + c16) * STRIDE + 16 * g + 4 * g4),
                                                                  *reinterpret_cast<const half4v *>(va + (16 * wr + c16) * STRIDE + 16 * g + 4 * g4), zero, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float x = t[v] + __uint_as_float(d[c][v]);
                        if ((__float_as_uint(x) & 0x7F800000u) == 0x7F800000u) S[c][v] = x;
                    }
                }
            }
            // (a NaN or an infinity would reach other outputs through the matrix instruction's zeros: a finite stand-in takes its place)
            auto finite = [](uint32_t x, int t) -> uint32_t {
                const uint32_t bound = (uint32_t)(15 + t + 1) << 10;                     // 2^(T + 1), above every element of the row
                half2v y = __builtin_elementwise_max(as_half2(x), as_half2((bound | 0x8000u) * 0x10001u));
                y = __builtin_elementwise_min(y, as_half2(bound * 0x10001u));
                return as_u32(y);
            };
            auto terms = [&](auto slow_c) {
            constexpr bool SLOW = decltype(slow_c)::value;
            // ---- terms: eight of each of a lane's products per matrix instruction, added up in the lane that owns the output ----
#pragma unroll 1
            for (int q = 0; q < L / 8; ++q) {
                uint32_t a[R][4];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(va + (16 * wr + 4 * g4 + r) * STRIDE + g * L + 8 * q);
                    a[r][0] = v.x; a[r][1] = v.y; a[r][2] = v.z; a[r][3] = v.w;
                    if constexpr (SLOW) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) a[r][w] = finite(a[r][w], pa.t_a);
                    }
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint4 bv = *reinterpret_cast<const uint4 *>(vb + ((wc * NC + c) * 16 + c16) * STRIDE + g * L + 8 * q);
                    uint32_t b[4] = {bv.x, bv.y, bv.z, bv.w};
                    if constexpr (SLOW) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) b[w] = finite(b[w], pa.t_b);
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        // (the four words side by side: a packed result is not ready for the next instruction)
                        half2v t[4];
#pragma unroll
                        for (int w = 0; w < 4; ++w) t[w] = as_half2(a[r][w]) * as_half2(b[w]);
#pragma unroll
                        for (int w = 0; w < 4; ++w) t[w] = t[w] * half2v{as_half2(sc[r][c])[0], as_half2(sc[r][c])[0]};
                        if constexpr (SLOW) {
#pragma unroll
                            for (int w = 0; w < 4; ++w) t[w] = t[w] * half2v{as_half2(sc[r][c])[1], as_half2(sc[r][c])[1]};
                        }
                        S[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(half8v{t[0][0], t[0][1], t[1][0], t[1][1], t[2][0], t[2][1], t[3][0], t[3][1]}, sel[r], S[c], 0, 0, 0);
                    }
                }
            }
            };
            if (__builtin_expect(slow, 0)) {
                terms(std::true_type{});
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) d[c][v] = packed_finish(pa, S[c][v] * 0x1p24f, em[c][v]);
            } else {
                terms(std::false_type{});
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) d[c][v] = packed_finish(pa, S[c][v], em[c][v] + (24u << 23));
            }
        }
    }
    // (a NaN travels with whatever pattern the arithmetic gives it; the model's is written once here)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if ((d[c][v] & 0x7FFFFFFFu) > 0x7F800000u) d[c][v] = pa.nan_bits;
    if (oi < m) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t j = out_col(c);
            if (wide) {
                if (j < n) *reinterpret_cast<uint4 *>(D + orow + j) = make_uint4(d[c][0], d[c][1], d[c][2], d[c][3]);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (j + v < n) D[orow + j + v] = d[c][v];
            }
        }
    }
}

// ---- host side ---------------------------------------------------------------------------

template <int TA, int TB, int WR, int WC, int NC, int L>
static mmaemu_status launch_packed_cfg(const PackedArgs &pa, const void *A, const void *B, const void *Cm, void *D, uint32_t m, uint32_t n,
                                       uint32_t k, uint64_t batch, hipStream_t s)
{
    constexpr uint32_t ROWS_A = 16 * WR, ROWS_B = 16 * WC * NC;
    const uint32_t bm = (m + ROWS_A - 1) / ROWS_A, bn = (n + ROWS_B - 1) / ROWS_B;
    const uint64_t blocks = batch * bm * bn;
    if (blocks > 0x7FFFFFFFull) { set_error("emulate_mma: too many blocks"); return MMAEMU_ERR_SHAPE; }
    const uint32_t remap = (blocks % 8 == 0 && blocks >= 64) ? 1u : 0u;
    hipLaunchKernelGGL((emulate_packed_kernel<TA, TB, WR, WC, NC, L>), dim3((uint32_t)blocks), dim3(64 * WR * WC), 0, s, pa, (const uint8_t *)A, (const uint8_t *)B,
                       (const uint32_t *)Cm, (uint32_t *)D, m, n, k, bm, bn, remap);
    MMAEMU_HIP(hipGetLastError());
    set_last_kernel("tiled %ux%u packed fp16 L=%d", ROWS_A, ROWS_B, L);
    return MMAEMU_OK;
}

// The side of the blocks that a problem is cut into, 64 or 32; 0 where neither grid has fewer than the 2^32 threads of one launch.
// A 64 x 64 block costs 0.47 (groups of 32) or 0.55 (groups of 16) of what the tiled kernels take for as many outputs, a 32 x 32 block
// 0.55 to 0.65 -- but both for the padding of edge blocks too, and 64 x 64 blocks need 2^21 outputs to keep all CUs busy.  So they
// are taken from there on where they pad at most a seventh more than 32 x 32 blocks do.  Groups of 32 on N(0,1) data, tiled
// kernel, 64 x 64, 32 x 32: 2^14 tiles of 32x32x64 162, 296, 100 us; 2^13 of 17x17x32 47, 85, 29; 512 of 65x65x64 50, 41, 29; 2^12 of
// 64x64x64 170, 80, 94; 2^12 of 33x33x32 98, 45, 58.  Groups of 16: 2^10 of 48x48x64 33 (in 16 x 16 blocks, which pad nothing), 27, 31.
static uint32_t packed_side(uint32_t m, uint32_t n, uint64_t batch)
{
    auto blocks = [&](uint64_t side) { return batch * ((m + side - 1) / side) * ((n + side - 1) / side); };
    const uint64_t large = blocks(64), small = blocks(32);
    if (batch * m * n >= (1ull << 21) && 7 * large <= 2 * small && large < (1ull << 32) / 512) return 64;
    return small < (1ull << 32) / 256 ? 32 : 0;
}

template <int TA, int TB>
static mmaemu_status launch_packed_types(const PackedArgs &pa, uint32_t L, const void *A, const void *B, const void *Cm, void *D, uint32_t m,
                                         uint32_t n, uint32_t k, uint64_t batch, hipStream_t s)
{
    const bool large = packed_side(m, n, batch) == 64;
    if constexpr (TA == TB) {
        if (L == 16) return large ? launch_packed_cfg<TA, TB, 4, 2, 2, 16>(pa, A, B, Cm, D, m, n, k, batch, s) : launch_packed_cfg<TA, TB, 2, 2, 1, 16>(pa, A, B, Cm, D, m, n, k, batch, s);
    }
    return large ? launch_packed_cfg<TA, TB, 4, 2, 2, 32>(pa, A, B, Cm, D, m, n, k, batch, s) : launch_packed_cfg<TA, TB, 2, 2, 1, 32>(pa, A, B, Cm, D, m, n, k, batch, s);
}

bool packed_takes(const ModelArgs &p, uint32_t ta, uint32_t tb, uint32_t m, uint32_t n, uint32_t k, uint64_t batch)
{
    if (p.c_mode != MMAEMU_C_IN_GROUP || p.skip_zero_terms || p.zero_result_positive || (p.flags & (FL_ACC16 | FL_NAN_PROPAGATE))) return false;
    // (two E5M2 rows span 64 places together, more than binary16 can scale: the tiled kernels)
    if (ta > MMAEMU_FP8_E5M2 || tb > MMAEMU_FP8_E5M2 || (ta == MMAEMU_FP8_E5M2 && tb == MMAEMU_FP8_E5M2)) return false;
    // (groups of 16: built for two E4M3 operands)
    if (!(p.L == 32 || (p.L == 16 && ta == tb)) || k % 32 != 0 || m <= 16 || n <= 16) return false;
    if (packed_side(m, n, batch) == 0) return false;
    // every sum an integer below 2^24; below F = 10 a row of E4M3 beside one of E5M2 (T = F - 17) would lose its smallest bits
    return p.F >= 10 && ((uint64_t)(p.L + 1) << (p.F + 2)) <= (1ull << 24);
}

mmaemu_status launch_emulate_packed(const ModelArgs &p, const void *A, const void *B, const void *Cm, void *D, uint32_t m, uint32_t n,
                                    uint32_t k, uint64_t batch, uint32_t ta, uint32_t tb, hipStream_t s)
{
    if (ta == MMAEMU_FP8_E5M2 && tb == MMAEMU_FP8_E5M2) { set_error("emulate_mma: the packed kernel takes no two E5M2 operands"); return MMAEMU_ERR_UNSUPPORTED; }
    PackedArgs pa = {};
    pa.F = p.F;
    pa.flags = p.flags;
    pa.out_mask = p.out_mask;
    pa.nan_bits = p.nan_bits;
    // The sum's unit is 2^-24, so the scaled products' maximum, top + x, may not lie below F - 24 (x >= -15 is also what the matrix
    // result holds), and one factor scales groups whose e_max (the accumulator joining) lies at F or below.  A row of E5M2 spans 32
    // places and needs T >= 8 to be held whole (E4M3: 17, T >= -7).
    pa.top = p.F - PACKED_ROOM;
    if (ta == tb) { pa.t_a = pa.top / 2; pa.t_b = pa.top - pa.t_a; }
    else if (ta == MMAEMU_FP8_E4M3) { pa.t_b = 8; pa.t_a = pa.top - 8; }
    else { pa.t_a = 8; pa.t_b = pa.top - 8; }
    pa.reach23 = (uint32_t)(16 + p.F - pa.top) << 23;
    pa.c2 = (254 + p.F - pa.top - 24) << 23;
    if (ta == MMAEMU_FP8_E5M2) return launch_packed_types<MMAEMU_FP8_E5M2, MMAEMU_FP8_E4M3>(pa, p.L, A, B, Cm, D, m, n, k, batch, s);
    return tb == MMAEMU_FP8_E4M3 ? launch_packed_types<MMAEMU_FP8_E4M3, MMAEMU_FP8_E4M3>(pa, p.L, A, B, Cm, D, m, n, k, batch, s)
                                 : launch_packed_types<MMAEMU_FP8_E4M3, MMAEMU_FP8_E5M2>(pa, p.L, A, B, Cm, D, m, n, k, batch, s);
}

} // namespace mmaemu

// Distribution of the deviation delta = D - D_real of a model's (or an instruction's) outputs from the real result
// (Sec. 6.2.4: the bias of the round-down modes shows as a distribution of delta shifted toward the negative side,
// against a symmetric one for the variant that truncates toward zero).  D_real = c + sum_k a_k b_k is taken exactly, and so is
// delta; only its binary64 image (for the three sums) is rounded.  Two ways: one thread sums an output's products (or four outputs'), adds D and
// subtracts that sum and the accumulator, in an unevaluated pair of binary64 numbers while that is exact and in a wide fixed-point
// number otherwise; whole tiles of FP16 and FP8 operands have their sums of products formed on the matrix cores (see there).  Linear bins of width 2^bin_exp
// around zero: bin i holds delta in [(i - 32) w, (i - 31) w), the outermost bins everything beyond.
#include "efdpa_pair.hpp"

namespace mmaemu {

constexpr int DEV_WORDS = sizeof(mmaemu_deviation_hist) / 8;
static_assert(DEV_WORDS == 5 + MMAEMU_DEVIATION_BINS + 3, "layout of mmaemu_deviation_hist");

__global__ void deviation_reset_kernel(mmaemu_deviation_hist *h)
{
    uint64_t *w = reinterpret_cast<uint64_t *>(h);
    if (threadIdx.x < DEV_WORDS) w[threadIdx.x] = 0ull;             // +0.0 is all-zero bits
}

// Elements kk .. kk + 7 of a row (bits as elem_bits gives them): `vec` says that the row's bytes from kk on are 16-byte
// aligned (8-byte for one-byte elements), so one or two wide loads bring them; per-element loads of 64 lanes, each in a
// row of its own, keep the address unit busy for longer than all the arithmetic of a sample takes.
__device__ __forceinline__ void load8(uint32_t t, uint32_t esize, const uint8_t *row, uint32_t kk, bool vec, uint32_t (&r)[8])
{
    if (!vec) {
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = elem_bits(t, esize, row, kk + q);
    } else if (esize == 2) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + 2u * kk);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) { r[2 * q] = w[q] & 0xFFFFu; r[2 * q + 1] = w[q] >> 16; }
    } else if (esize == 1) {
        const uint2 v = *reinterpret_cast<const uint2 *>(row + kk);
#pragma unroll
        for (int q = 0; q < 4; ++q) { r[q] = (v.x >> (8 * q)) & 0xFFu; r[4 + q] = (v.y >> (8 * q)) & 0xFFu; }
    } else {
        const uint4 v0 = *reinterpret_cast<const uint4 *>(row + 4u * kk), v1 = *reinterpret_cast<const uint4 *>(row + 4u * kk + 16u);
        const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = t == MMAEMU_TF32 ? w[q] >> 13 : w[q];
    }
}

// The same through the wide fixed-point number (exact for any finite operands): sign, whether delta is zero,
// floor(delta / 2^bin_exp) clamped to +-NB, and |delta|'s binary64 image (its 64 bits from the leading one downward,
// converted once).
__device__ __noinline__ void delta_wide(DynFmt fa, DynFmt fb, const uint8_t *a, const uint8_t *b, uint32_t k, uint32_t cb, uint32_t db,
                                        int unit_bit, uint32_t &neg, bool &zero, int &fi, double &ad)
{
    constexpr int NB = MMAEMU_DEVIATION_BINS;
    uint32_t w[XL];
    for (int q = 0; q < XL; ++q) w[q] = 0u;
    for (uint32_t kk = 0; kk < k; ++kk) {
        const Dec x = decode_as(fa, fa.load(a, kk), 0u), y = decode_as(fb, fb.load(b, kk), 0u);
        wide_add(w, sig_product(fa, fb, x, y), x.exp + y.exp - fa.mb() - fb.mb(), (x.sign ^ y.sign) ^ 1u);   // - a b
    }
    {
        const uint32_t Ec = (cb >> 23) & 0xFFu, Ed = (db >> 23) & 0xFFu;
        wide_add(w, (cb & 0x7FFFFFu) | (Ec ? 0x800000u : 0u), (int)(Ec ? Ec : 1u) - 150, (cb >> 31) ^ 1u);        // - c
        wide_add(w, (db & 0x7FFFFFu) | (Ed ? 0x800000u : 0u), (int)(Ed ? Ed : 1u) - 150, db >> 31);               // + D
    }
    neg = w[XL - 1] >> 31;
    if (neg) {
        uint32_t carry = 1;
        for (int q = 0; q < XL; ++q) {
            const uint64_t t = (uint64_t)(~w[q]) + carry;
            w[q] = (uint32_t)t;
            carry = (uint32_t)(t >> 32);
        }
    }
    int top = XL - 1;
    while (top >= 0 && w[top] == 0u) --top;
    zero = top < 0;
    fi = 0;
    ad = 0.0;
    if (zero) return;
    const int hi_bit = 32 * top + (31 - __builtin_clz(w[top]));
    // floor(delta / 2^bin_exp) from the magnitude: its bits from unit_bit upward, and whether anything lies below
    if (hi_bit < unit_bit) fi = neg ? -1 : 0;
    else if (hi_bit - unit_bit >= 6) fi = neg ? -NB : NB;
    else {
        const int limb = unit_bit >> 5, off = unit_bit & 31;
        uint32_t v = w[limb] >> off;
        if (off && limb + 1 < XL) v |= w[limb + 1] << (32 - off);
        const int q = (int)(v & 63u);
        bool below = (off != 0) && (w[limb] & ((1u << off) - 1u)) != 0u;
        for (int t = 0; t < limb; ++t) below |= w[t] != 0u;
        fi = neg ? (below ? -q - 1 : -q) : q;
    }
    const int low_bit = hi_bit - 63;
    uint64_t mag;
    int lsb;
    if (low_bit <= 0) { mag = ((uint64_t)w[1] << 32) | w[0]; lsb = XBASE; }
    else {
        const int l0 = low_bit >> 5, sh = low_bit & 31;
        const uint32_t a0 = w[l0], a1 = w[l0 + 1], a2 = (l0 + 2 < XL) ? w[l0 + 2] : 0u;
        const u128 win = ((u128)a2 << 64) | ((u128)a1 << 32) | a0;
        mag = (uint64_t)(win >> sh);
        lsb = XBASE + low_bit;
    }
    ad = ldexp((double)mag, lsb);
}

// sign, whether delta is zero, floor(delta / 2^bin_exp) clamped to +-NB and |delta|'s binary64 image, from a pair that holds delta
__device__ __forceinline__ void place_pair(const ExactPair &pr, int bin_exp, uint32_t &neg, bool &zero, int &fi, double &ad)
{
    constexpr int NB = MMAEMU_DEVIATION_BINS;
    double h, l;
    two_sum(pr.hi, pr.lo, h, l);                                     // h = RN(delta), l = delta - h
    neg = h < 0.0;
    zero = h == 0.0;
    ad = __builtin_fabs(h);
    // floor(delta / 2^bin_exp): of h, and one less where h is a whole number of bins and l lies below it (a
    // fractional h / w keeps at least one of its own last places to either side, more than |l / w|)
    const double qh = ldexp(h, -bin_exp);
    if (qh >= (double)NB) fi = NB;
    else if (qh <= -(double)NB) fi = -NB;
    else if (qh == 0.0) fi = neg ? -1 : 0;                           // (h / w below the binary64 range)
    else {
        const double fl = __builtin_floor(qh);
        fi = (int)fl - ((fl == qh && l < 0.0) ? 1 : 0);
    }
}

// Eight elements of one row as binary32 values (NaN and infinities as themselves), one branch on the type for all
__device__ __forceinline__ void elem_floats8(uint32_t t, const uint32_t (&bits)[8], float (&v)[8])
{
    auto all = [&](auto type_tag) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            uint32_t ex;
            bool wild = false;
            decode_elem<decltype(type_tag)::value>(bits[q], 0u, 0u, v[q], ex, wild);
        }
    };
    switch (t) {   // uniform
    case MMAEMU_FP8_E4M3: all(std::integral_constant<int, MMAEMU_FP8_E4M3>{}); break;
    case MMAEMU_FP8_E5M2: all(std::integral_constant<int, MMAEMU_FP8_E5M2>{}); break;
    case MMAEMU_FP6_E2M3: all(std::integral_constant<int, MMAEMU_FP6_E2M3>{}); break;
    case MMAEMU_FP6_E3M2: all(std::integral_constant<int, MMAEMU_FP6_E3M2>{}); break;
    case MMAEMU_FP4_E2M1: all(std::integral_constant<int, MMAEMU_FP4_E2M1>{}); break;
    case MMAEMU_FP16: all(std::integral_constant<int, MMAEMU_FP16>{}); break;
    default: all(std::integral_constant<int, MMAEMU_BF16>{}); break;
    }
}

// The products' sum of FP16, FP8, FP6 and FP4 operands in two binary64 numbers: every product is a multiple of 2^-48 below
// 2^32 in magnitude, so adding and taking away a constant whose last place is 2^-8 splits it there; the upper parts are
// multiples of 2^-8 that stay below 2^45 and the lower ones multiples of 2^-48 below 2^4 for k up to SPLIT_MAX_K: both
// sums are exact.  An infinite or NaN operand leaves a NaN in the lower sum.
constexpr uint32_t SPLIT_MAX_K = 8192;
struct SplitSum {
    double upper = 0.0, lower = 0.0;
    __device__ __forceinline__ void add(float x, float y)
    {
        constexpr double M = 0x1.8p+44;
        const double p = (double)(x * y);                            // exact: 22 significant bits
        const double u = (p + M) - M;
        upper += u;
        lower += p - u;
    }
};
__host__ __device__ constexpr bool splits(uint32_t t)
{
    return t == MMAEMU_FP16 || t == MMAEMU_FP8_E4M3 || t == MMAEMU_FP8_E5M2 || t == MMAEMU_FP6_E2M3 || t == MMAEMU_FP6_E3M2 || t == MMAEMU_FP4_E2M1;
}

// One thread per W consecutive outputs of a row (W = 4: every output sampled, n a multiple of 4, many outputs; else one sample each).
// SPLIT: products summed as SplitSum does (7 vector instructions per term), only D, the accumulator and the two sums go
// through the pair of binary64 numbers; else (BF16: hundreds of binary places, or k beyond SPLIT_MAX_K) every product does
// (15 per term).  With one output per thread, all through the pair, checks per element, 64-bit divisions per sample and three
// LDS atomics per sample on few addresses, 2^24 outputs of 32x32x8 FP16 tiles took 229 us, so 119 (bound by binary64 issue; whole tiles have a kernel of their own below).
template <int W, bool SPLIT>
__global__ void __launch_bounds__(256)
deviation_kernel(const void *__restrict__ A, const void *__restrict__ B, const uint32_t *__restrict__ C,
                 const uint32_t *__restrict__ D, uint32_t m, uint32_t n, uint32_t k, uint32_t ta, uint32_t tb, uint64_t stride,
                 uint64_t nitems, int bin_exp, mmaemu_deviation_hist *hist)
{
    constexpr int NB = MMAEMU_DEVIATION_BINS, COPIES = 8;
    __shared__ uint32_t counts[5], bins[NB][COPIES];                 // (lanes of a wavefront spread over copies: most samples share few bins)
    if (threadIdx.x < 5) counts[threadIdx.x] = 0u;
    for (uint32_t i = threadIdx.x; i < NB * COPIES; i += 256) (&bins[0][0])[i] = 0u;
    __syncthreads();
    const DynFmt fa = dyn_fmt(ta), fb = dyn_fmt(tb);
    const uint32_t esa = (uint32_t)fa.width_ / 8u, esb = (uint32_t)fb.width_ / 8u;
    const uint64_t per_tile = (uint64_t)m * n;
    const int unit_bit = bin_exp - XBASE;                            // index of the bit that weighs one bin width
    const bool vec_a = (reinterpret_cast<uintptr_t>(A) & 15u) == 0 && k % 8u == 0, vec_b = (reinterpret_cast<uintptr_t>(B) & 15u) == 0 && k % 8u == 0;
    const double finite_max = 0x1.fffffffffffffp+1023;
    double sum = 0.0, sum_abs = 0.0, sum_sq = 0.0;
    uint32_t n_seen = 0, n_bad = 0, n_neg = 0, n_zero = 0;
    // (a workgroup handles at most 2^31 samples: the 32-bit counters cannot overflow, see the launch)
    for (uint64_t item = (uint64_t)blockIdx.x * 256u + threadIdx.x; item < nitems; item += (uint64_t)gridDim.x * 256u) {
        const uint64_t o = W == 1 ? item * stride : item * (uint64_t)W;
        uint64_t tile;
        uint32_t rem;
        if ((o >> 32) == 0 && (per_tile >> 32) == 0) {               // (a 64-bit division costs a hundred instructions)
            const uint32_t q = (uint32_t)o / (uint32_t)per_tile;
            tile = q;
            rem = (uint32_t)o - q * (uint32_t)per_tile;
        } else {
            tile = o / per_tile;
            rem = (uint32_t)(o - tile * per_tile);
        }
        const uint32_t i = rem / n, j = rem - i * n;
        const uint8_t *a = static_cast<const uint8_t *>(A) + (tile * m + i) * (uint64_t)k * esa;
        const uint8_t *b = static_cast<const uint8_t *>(B) + (tile * n + j) * (uint64_t)k * esb;
        uint32_t cb[W], db[W];
        if constexpr (W == 4) {
            const uint4 d4 = *reinterpret_cast<const uint4 *>(D + o), c4 = C ? *reinterpret_cast<const uint4 *>(C + o) : make_uint4(0u, 0u, 0u, 0u);
            db[0] = d4.x; db[1] = d4.y; db[2] = d4.z; db[3] = d4.w;
            cb[0] = c4.x; cb[1] = c4.y; cb[2] = c4.z; cb[3] = c4.w;
        } else {
            cb[0] = C ? C[o] : 0u;
            db[0] = D[o];
        }
        // delta as an unevaluated pair of binary64 numbers (efdpa_pair.hpp): D, then the products and the accumulator taken
        // away; while the pair holds the sum exactly (always for FP16 / FP8 operands; BF16 operands spread over hundreds of
        // binary places may leave it) sign, bin and binary64 image follow from the normalised pair
        ExactPair pr[W];
        bool bad[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            bad[w] = (cb[w] & 0x7F800000u) == 0x7F800000u || (db[w] & 0x7F800000u) == 0x7F800000u;
            pr[w].start(db[w]);
        }
        if constexpr (SPLIT) {
            SplitSum sp[W];
            uint32_t kk = 0;
            for (; kk + 8 <= k; kk += 8) {
                uint32_t raw[8];
                float xa[8], xb[8];
                load8(ta, esa, a, kk, vec_a, raw);
                elem_floats8(ta, raw, xa);
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    load8(tb, esb, b + (uint64_t)w * k * esb, kk, vec_b, raw);
                    elem_floats8(tb, raw, xb);
#pragma unroll
                    for (int q = 0; q < 8; ++q) sp[w].add(xa[q], xb[q]);
                }
            }
            for (; kk < k; ++kk) {
                const float x = (float)elem_value(ta, elem_bits(ta, esa, a, kk), 0u);
#pragma unroll
                for (int w = 0; w < W; ++w) sp[w].add(x, (float)elem_value(tb, elem_bits(tb, esb, b + (uint64_t)w * k * esb, kk), 0u));
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                bad[w] |= !(__builtin_fabs(sp[w].lower) <= finite_max);
                // (hi + lo = D - upper exactly; the lower sum joins lo, and what lo cannot hold shows in `lost`, a sum of
                // magnitudes: the accumulator below cannot cancel it)
                double residue;
                two_sum(pr[w].hi, -sp[w].upper, pr[w].hi, pr[w].lo);
                two_sum(pr[w].lo, -sp[w].lower, pr[w].lo, residue);
                pr[w].lost = __builtin_fabs(residue);
            }
        } else {
            // (T: the type of both operands where it is known when the loop is compiled, else -1.  With the branches on the type
            // inside the loop few wavefronts wait for them: 64x64x4096 in BF16 476 us with, 306 us without)
            uint32_t kk = 0;
            auto eights = [&](auto type_c) {
                constexpr int T = decltype(type_c)::value;
                const uint32_t t_a = T < 0 ? ta : (uint32_t)T, t_b = T < 0 ? tb : (uint32_t)T, es_a = T < 0 ? esa : 2u, es_b = T < 0 ? esb : 2u;
                for (; kk + 8 <= k; kk += 8) {
                    // (eight elements of each row fetched before the first is used: one wait per eight terms)
                    uint32_t ra[8], rb[8];
                    load8(t_a, es_a, a, kk, vec_a, ra);
                    load8(t_b, es_b, b, kk, vec_b, rb);
                    double xa[8], xb[8];
                    elem_values(t_a, ra, 0u, xa);                        // (one branch on the type per eight elements)
                    elem_values(t_b, rb, 0u, xb);
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        bad[0] |= !(__builtin_fabs(xa[q]) <= finite_max) || !(__builtin_fabs(xb[q]) <= finite_max);
                        pr[0].add(-xa[q], xb[q]);
                    }
                }
            };
            if (ta == MMAEMU_BF16 && tb == MMAEMU_BF16) eights(std::integral_constant<int, MMAEMU_BF16>{});
            else if (ta == MMAEMU_FP16 && tb == MMAEMU_FP16) eights(std::integral_constant<int, MMAEMU_FP16>{});
            else eights(std::integral_constant<int, -1>{});
            for (; kk < k; ++kk) {
                const double x = elem_value(ta, elem_bits(ta, esa, a, kk), 0u), y = elem_value(tb, elem_bits(tb, esb, b, kk), 0u);
                bad[0] |= !(__builtin_fabs(x) <= finite_max) || !(__builtin_fabs(y) <= finite_max);
                pr[0].add(-x, y);
            }
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (bad[w]) { ++n_bad; continue; }
            pr[w].add(-(double)__uint_as_float(cb[w]), 1.0);
            uint32_t neg;
            bool zero;
            int fi;
            double ad;
            if (pr[w].lost == 0.0) {
                place_pair(pr[w], bin_exp, neg, zero, fi, ad);
            } else {
                delta_wide(fa, fb, a, b + (uint64_t)w * k * esb, k, cb[w], db[w], unit_bit, neg, zero, fi, ad);
            }
            ++n_seen;
            n_zero += zero ? 1u : 0u;
            n_neg += (!zero && neg) ? 1u : 0u;
            int bin = zero ? NB / 2 : fi + NB / 2;
            bin = bin < 0 ? 0 : (bin > NB - 1 ? NB - 1 : bin);
            atomicAdd(&bins[bin][threadIdx.x % COPIES], 1u);
            ad = zero ? 0.0 : ad;
            sum += neg ? -ad : ad;
            sum_abs += ad;
            sum_sq += ad * ad;
        }
    }
    // the counts and the three sums: over the wavefront by lane exchanges, over the workgroup through LDS, then one atomic per
    // workgroup and word (thousands of wavefronts adding to the same few words took longer than everything else in the kernel)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        sum += __shfl_xor(sum, off, 64);
        sum_abs += __shfl_xor(sum_abs, off, 64);
        sum_sq += __shfl_xor(sum_sq, off, 64);
        n_seen += __shfl_xor(n_seen, off, 64);
        n_bad += __shfl_xor(n_bad, off, 64);
        n_neg += __shfl_xor(n_neg, off, 64);
        n_zero += __shfl_xor(n_zero, off, 64);
    }
    __shared__ double wave_sums[4][3];
    if ((threadIdx.x & 63u) == 0u) {
        wave_sums[threadIdx.x >> 6][0] = sum;
        wave_sums[threadIdx.x >> 6][1] = sum_abs;
        wave_sums[threadIdx.x >> 6][2] = sum_sq;
        const uint32_t c5[5] = {n_seen, n_bad, n_neg, n_zero, n_seen - n_neg - n_zero};
#pragma unroll
        for (int q = 0; q < 5; ++q) if (c5[q]) atomicAdd(&counts[q], c5[q]);
    }
    __syncthreads();
    double *gd = reinterpret_cast<double *>(reinterpret_cast<uint64_t *>(hist) + 5 + NB);
    unsigned long long *gc = reinterpret_cast<unsigned long long *>(hist);
    if (threadIdx.x < 3) {
        const double t = (wave_sums[0][threadIdx.x] + wave_sums[1][threadIdx.x]) + (wave_sums[2][threadIdx.x] + wave_sums[3][threadIdx.x]);
        if (t != 0.0) atomicAdd(&gd[threadIdx.x], t);
    } else if (threadIdx.x >= 64u && threadIdx.x < 64u + 5u) {
        if (counts[threadIdx.x - 64u]) atomicAdd(gc + (threadIdx.x - 64u), (unsigned long long)counts[threadIdx.x - 64u]);
    } else if (threadIdx.x >= 128u && threadIdx.x < 128u + NB) {
        const uint32_t bin = threadIdx.x - 128u;
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < COPIES; ++q) t += bins[bin][q];
        if (t) atomicAdd(gc + 5 + bin, (unsigned long long)t);
    }
}

// ---- whole tiles of FP16 and FP8 operands: the products' sums on the matrix cores -------------
//
// A wavefront owns 16 x 16 CB outputs of a tile and forms their sums of products with v_mfma_f64_16x16x4_f64, a chain of fused
// multiply-adds that is exact while every product is a multiple of one unit and the sums stay below 2^53 of them.  The types alone may
// guarantee that (E4M3 x E4M3); else the wavefront takes the largest and the smallest exponent of its rows' elements.  An output's end
// is four binary64 operations, with four comparisons that say whether they were exact: D - S first, which cancels, then the
// accumulator.  Outputs for which they were not follow one after the other, an output of all lanes at a time, as expansions of
// binary64 numbers, exact for all finite ones: accumulators of 2^30 (some 53 places above the products' unit) or of any exponent 95 us where
// the others take 38 (2^24 outputs of 32x32x8 FP16; the kernel of four outputs per thread 115 and 2150).  With the expansion beside every
// output's end they took 68, but the others 39.
// Where the exponents lie too far apart the wavefront splits every element at 2^-4 into two parts, whose sums of products are exact up
// to SPLIT_MAX_K, and every output's sum is two numbers.
// Bound: HBM (C and D are read once, 8 bytes per output): 2^24 outputs of 32x32x8 FP16 tiles 114 -> 47 us (3.2 TB/s).  Blocks of 32 rows
// took 54: fewer wavefronts to hide the loads behind; 256, 1024 and 2048 workgroups for 512 took 55, 48 and 62 (each ends in
// atomics on the same lines).
constexpr int TILE_COPIES = 32, TILE_BINS = MMAEMU_DEVIATION_BINS + 1;     // (the last row takes what is not counted, modulo 2^32)
// Workgroups, and as many more beyond 2^40 samples that none counts more than 2^31 (a sum of 64 bits at its end, over copies of which
// none could wrap, cost a launch 0.7 us).
constexpr uint64_t MAX_SAMPLES = 1ull << 43, TILE_WORKGROUPS = 512, TILE_WORKGROUPS_MANY = 4096;
static_assert((1ull << 40) / TILE_WORKGROUPS <= 1ull << 31 && MAX_SAMPLES / TILE_WORKGROUPS_MANY <= 1ull << 31, "counters of a workgroup");

struct DevTileArgs {
    const uint8_t *A, *B;
    const uint32_t *C, *D;
    uint32_t m, n, k, ta, tb, stride;
    int32_t bin_exp, slack;             // slack: how far apart the exponents may lie (see the launch)
    uint32_t exact_types, bm, bn;
    uint64_t nitems;
};

// two consecutive elements of a row as they lie in memory, and as binary32 values (FP8: whether E5M2)
template <bool FP8> __device__ __forceinline__ uint32_t pair_load(const uint8_t *p)
{
    if constexpr (FP8) return *reinterpret_cast<const uint16_t *>(p);
    else return *reinterpret_cast<const uint32_t *>(p);
}
template <bool FP8> __device__ __forceinline__ void pair_values(bool e5m2, uint32_t w, float (&v)[2])
{
    if constexpr (FP8) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 x = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), y = __builtin_amdgcn_cvt_pk_f32_bf8((int)w, false);
        v[0] = e5m2 ? y.x : x.x; v[1] = e5m2 ? y.y : x.y;
    } else {
        typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
        const f16x2 h = __builtin_bit_cast(f16x2, w);
        v[0] = (float)h[0]; v[1] = (float)h[1];
    }
}

// largest magnitude pattern and (less one, zeros left out) smallest of a lane's elements
struct Span {
    uint32_t most = 0u, least = 0xFFFFFFFFu;
    __device__ __forceinline__ void take(const float (&v)[2])
    {
        const uint32_t u0 = __float_as_uint(v[0]) & 0x7FFFFFFFu, u1 = __float_as_uint(v[1]) & 0x7FFFFFFFu;
        most = max(max(u0, u1), most);
        least = min(min(u0 - 1u, u1 - 1u), least);
    }
    // exponent fields over the wavefront: the largest in the low half, 511 less the smallest in the high half (256 where all are zero)
    __device__ __forceinline__ uint32_t wave() const
    {
        const uint32_t lo = least == 0xFFFFFFFFu ? 255u : (least + 1u) >> 23;
        uint32_t x = (most >> 23) | ((511u - lo) << 16);
#if defined(__HIP_DEVICE_COMPILE__)
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false));
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false));
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false));
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false));
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
        x = pk_max_u16(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
        x = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
#endif
        return x;
    }
};

// delta = d - s - low - c (finite; low only where LOW) exactly, as an expansion: h, delta rounded once, and q, floor(delta / 2^bin_exp).  One
// summand after the other goes through the parts so far from the smallest upward, which leaves parts that do not overlap (Shewchuk 1997);
// on the way down again they become h and remainders, of which the first that is not zero has the sign of delta - h.
template <bool LOW>
__device__ __forceinline__ void place_expansion(double d, double s, double low, double c, int bin_exp, double &h, double &q)
{
    double e0 = 0.0, e1, e2, e3, t, u;
    two_sum(d, -s, u, t);
    if constexpr (LOW) {
        double f1, f2;
        two_sum(t, -low, t, e0);
        two_sum(u, t, f2, f1);
        two_sum(e0, -c, t, e0);
        two_sum(f1, t, t, e1);
        two_sum(f2, t, e3, e2);
    } else {
        two_sum(t, -c, t, e1);
        two_sum(u, t, e3, e2);
    }
    double r1, r2, r3, r4;
    two_sum(e3, e2, e3, r1);
    two_sum(r1, e1, r2, r3);
    two_sum(e3, r2, h, r4);
    double rest = r4 != 0.0 ? r4 : r3;
    if constexpr (LOW) {
        two_sum(r3, e0, t, r3);
        two_sum(r4, t, t, r4);
        two_sum(h, t, h, rest);
        rest = rest != 0.0 ? rest : (r4 != 0.0 ? r4 : r3);
    }
    const double qh = ldexp(h, -bin_exp);
    q = __builtin_floor(qh);
    if (q == qh && rest < 0.0) q -= 1.0;                                 // (a fractional h / w lies further from the next whole number)
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// What a lane sums up and what its wavefront counts.  `bin` NB: not counted (h is zero then).
struct DevTally {
    double sum = 0.0, sum_abs = 0.0, sum_sq = 0.0;
    uint32_t neg = 0, zero = 0, out = 0, bad = 0;                       // out: not sampled; bad: skipped (both come with h = 0)
    __device__ __forceinline__ void take(double h, uint32_t bin, uint32_t lane, uint32_t *bins)
    {
        neg += (uint32_t)__popcll(__ballot(h < 0.0));
        zero += (uint32_t)__popcll(__ballot(h == 0.0));
        atomicAdd(&bins[bin * TILE_COPIES + (lane & (TILE_COPIES - 1))], 1u);
        sum += h;
        sum_abs += __builtin_fabs(h);
        sum_sq = __builtin_fma(h, h, sum_sq);
    }
};

template <bool FP8, int CB, bool STRIDED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
deviation_tile_kernel(DevTileArgs g, mmaemu_deviation_hist *hist)
{
    constexpr int NB = MMAEMU_DEVIATION_BINS;
    __shared__ uint32_t bins[TILE_BINS * TILE_COPIES];
    for (uint32_t i = threadIdx.x; i < TILE_BINS * TILE_COPIES; i += 512) bins[i] = 0u;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t c16 = lane & 15u, g4 = lane >> 4;
    constexpr uint32_t ES = FP8 ? 1u : 2u;
    const bool a5 = g.ta == MMAEMU_FP8_E5M2, b5 = g.tb == MMAEMU_FP8_E5M2;
    const uint32_t *const acc = g.C ? g.C : g.D;                       // (without an accumulator D is read again, and masked)
    const uint32_t acc_mask = g.C ? 0xFFFFFFFFu : 0u;
    const f64x4 zero4 = {0.0, 0.0, 0.0, 0.0};
    const uint32_t lane_mod = STRIDED ? (g4 * g.n + CB * c16) % g.stride : 0u;
    DevTally tally;
    unsigned long long seen = 0, skipped = 0, negative = 0, none = 0;          // (of the wavefront; none: zero)
    for (uint64_t item = (uint64_t)blockIdx.x * 8u + wave; item < g.nitems; item += (uint64_t)gridDim.x * 8u) {
        uint64_t tile; uint32_t rem;
        split_item(item, g.bm * g.bn, tile, rem);
        const uint32_t i0 = (rem / g.bn) * 16, j0 = (rem % g.bn) * (16 * CB);
        const uint64_t row_a = tile * g.m + i0 + c16, row_b = tile * g.n + j0 + CB * c16;
        const uint8_t *pa = g.A + (row_a * g.k + 2u * g4) * ES, *pb = g.B + (row_b * g.k + 2u * g4) * ES;
        const uint64_t out_row = tile * g.m + i0 + g4;                         // rows out_row + 4 v, columns j0 + CB c16 + c
        const uint64_t o0 = out_row * g.n + j0 + CB * c16;
        uint32_t o0_mod = 0;
        if constexpr (STRIDED) {
            o0_mod = (uint32_t)(((tile * g.m + i0) * g.n + j0) % g.stride) + lane_mod;
            o0_mod -= o0_mod >= g.stride ? g.stride : 0u;
        }
        auto sampled = [&](int v, int c) -> bool {
            if constexpr (!STRIDED) return true;
            const uint32_t x = o0_mod + ((uint32_t)(4 * v) * g.n + c) % g.stride;      // (the output's index modulo stride, or that and stride)
            return x == 0u || x == g.stride;
        };
        uint32_t db[4][CB], cb[4][CB];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const uint64_t o = o0 + (uint64_t)(4 * v) * g.n;
            if constexpr (CB == 2) {
                const uint2 d2 = *reinterpret_cast<const uint2 *>(g.D + o), c2 = *reinterpret_cast<const uint2 *>(acc + o);
                db[v][0] = d2.x; db[v][CB - 1] = d2.y; cb[v][0] = c2.x & acc_mask; cb[v][CB - 1] = c2.y & acc_mask;
            } else {
                db[v][0] = g.D[o];
                cb[v][0] = acc[o] & acc_mask;
            }
        }
        f64x4 S[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) S[c] = zero4;
        Span span_a, span_b;
        uint32_t wa, wb[CB];
        auto fetch = [&](uint32_t k0) {
            wa = pair_load<FP8>(pa + (uint64_t)k0 * ES);
#pragma unroll
            for (int c = 0; c < CB; ++c) wb[c] = pair_load<FP8>(pb + ((uint64_t)c * g.k + k0) * ES);
        };
        fetch(0);
#pragma unroll 1
        for (uint32_t k0 = 0; k0 < g.k; k0 += 8) {
            float a[2], b[CB][2];
            pair_values<FP8>(a5, wa, a);
            span_a.take(a);
#pragma unroll
            for (int c = 0; c < CB; ++c) { pair_values<FP8>(b5, wb[c], b[c]); span_b.take(b[c]); }
            if (k0 + 8 < g.k) fetch(k0 + 8);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < CB; ++c) S[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[h], (double)b[c][h], S[c], 0, 0, 0);
        }
        bool split = false;
        if (!g.exact_types) {
            const uint32_t xa = span_a.wave(), xb = span_b.wave();
            // (an infinite or NaN element, whose field is 255, goes on split)
            split = (int)((xa & 0xFFFFu) + (xa >> 16) + (xb & 0xFFFFu) + (xb >> 16)) - 2 * 511 > g.slack || (xa & 0xFFFFu) == 255u || (xb & 0xFFFFu) == 255u;
        }
        tally.neg = tally.zero = tally.out = tally.bad = 0;
        uint32_t open = 0;                                            // outputs whose end was not exact, bit v CB + c; 0 where split
        // one output's end; LOW: the products' sum is s + low
        auto end = [&](auto low_c, int i, uint32_t dbits, uint32_t cbits, double s, double low, bool in) {
            constexpr bool LOW = decltype(low_c)::value;
            const double dd = (double)__uint_as_float(dbits), cc = (double)__uint_as_float(cbits);
            // (a difference is exact where adding it to the one, and taking it from the other, operand gives the operands back;
            // false for NaN)
            double r1 = dd - s;
            bool exact = (r1 + s == dd) & (dd - r1 == s);
            if constexpr (LOW) {
                const double r0 = r1;
                r1 = r0 - low;
                exact = exact & (r1 + low == r0) & (r0 - r1 == low);
            }
            double h = r1 - cc;
            exact = exact & (h + cc == r1) & (r1 - h == cc);
            double q = __builtin_floor(ldexp(h, -g.bin_exp));
            const bool counted = in & exact;
            if (__any(in && !exact)) {
                // (none of the finite ones overflows, so that h is finite exactly where everything is)
                const bool finite = __builtin_fabs(h) <= 0x1.fffffffffffffp+1023;
                if (in && !exact && finite) open |= 1u << i;
                const uint32_t skip = (uint32_t)__popcll(__ballot(in && !finite));
                tally.bad += skip;
                tally.out -= skip;
            }
            q = __builtin_fmax(__builtin_fmin(q, (double)(NB / 2 - 1)), (double)(-NB / 2));
            const uint32_t bin = (uint32_t)((int)q + NB / 2);
            tally.out += (uint32_t)__popcll(__ballot(!counted));
            tally.take(counted ? h : 0.0, counted ? bin : (uint32_t)NB, lane, bins);
        };
        // the end of an output of the lanes' as an expansion (row 4 v of theirs)
        auto settle = [&](auto low_c, int v, int c, double s, double low, bool mine) {
            constexpr bool LOW = decltype(low_c)::value;
            const uint64_t o = o0 + (uint64_t)(4 * v) * g.n + c;
            double h, q;
            place_expansion<LOW>((double)__uint_as_float(g.D[o]), s, low, (double)__uint_as_float(acc[o] & acc_mask), g.bin_exp, h, q);
            q = __builtin_fmax(__builtin_fmin(q, (double)(NB / 2 - 1)), (double)(-NB / 2));
            seen += 64u;
            tally.out += (uint32_t)__popcll(__ballot(!mine));
            tally.take(mine ? h : 0.0, mine ? (uint32_t)((int)q + NB / 2) : (uint32_t)NB, lane, bins);
        };
        seen += 64u * 4 * CB;
        if (__builtin_expect(!split, 1)) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int c = 0; c < CB; ++c) end(std::false_type{}, v * CB + c, db[v][c], cb[v][c], S[c][v], 0.0, sampled(v, c));
            if (__builtin_expect(__any(open != 0u), 0)) {
#pragma unroll 1
                for (int i = 0; i < 4 * CB; ++i) {
                    if (!__any((open >> i) & 1u)) continue;
                    double sum = 0.0;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int c = 0; c < CB; ++c) sum = i == v * CB + c ? S[c][v] : sum;
                    settle(std::false_type{}, i / CB, i % CB, sum, 0.0, ((open >> i) & 1u) != 0u);
                }
            }
        } else {
#pragma unroll 1
            for (int c = 0; c < CB; ++c) {
                f64x4 H = zero4, M = zero4, L = zero4;
                const uint8_t *const qb = pb + (uint64_t)c * g.k * ES;
                uint32_t xa = pair_load<FP8>(pa), xb = pair_load<FP8>(qb);
#pragma unroll 1
                for (uint32_t k0 = 0; k0 < g.k; k0 += 8) {
                    float a[2], b[2];
                    pair_values<FP8>(a5, xa, a);
                    pair_values<FP8>(b5, xb, b);
                    if (k0 + 8 < g.k) { xa = pair_load<FP8>(pa + (k0 + 8) * ES); xb = pair_load<FP8>(qb + (k0 + 8) * ES); }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        constexpr float CUT = 0x1.8p+19f;              // (its last place is 2^-4)
                        const float ah = (a[h] + CUT) - CUT, bh = (b[h] + CUT) - CUT;
                        const double al = (double)(a[h] - ah), bl = (double)(b[h] - bh);
                        H = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ah, (double)bh, H, 0, 0, 0);
                        M = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ah, bl, M, 0, 0, 0);
                        M = __builtin_amdgcn_mfma_f64_16x16x4f64(al, (double)bh, M, 0, 0, 0);
                        L = __builtin_amdgcn_mfma_f64_16x16x4f64(al, bl, L, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double hi, lo;
                    two_sum(H[v], M[v], hi, lo);
                    lo += L[v];                                        // (exact: below 2^4, a multiple of 2^-48)
                    const uint64_t o = o0 + (uint64_t)(4 * v) * g.n + c;
                    open = 0;
                    end(std::true_type{}, 0, g.D[o], acc[o] & acc_mask, hi, lo, sampled(v, c));
                    if (__builtin_expect(__any(open != 0u), 0)) settle(std::true_type{}, v, c, hi, lo, open != 0u);
                }
            }
        }
        seen -= tally.out + tally.bad;
        skipped += tally.bad;
        negative += tally.neg;
        none += (unsigned long long)tally.zero - tally.out - tally.bad;
    }
    // one atomic per workgroup and word
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        tally.sum += __shfl_xor(tally.sum, off, 64);
        tally.sum_abs += __shfl_xor(tally.sum_abs, off, 64);
        tally.sum_sq += __shfl_xor(tally.sum_sq, off, 64);
    }
    __shared__ double wave_sums[8][3];
    __shared__ unsigned long long wave_counts[8][5];
    if (lane == 0) {
        wave_sums[wave][0] = tally.sum; wave_sums[wave][1] = tally.sum_abs; wave_sums[wave][2] = tally.sum_sq;
        wave_counts[wave][0] = seen; wave_counts[wave][1] = skipped; wave_counts[wave][2] = negative; wave_counts[wave][3] = none;
        wave_counts[wave][4] = seen - negative - none;
    }
    __syncthreads();
    unsigned long long *gc = reinterpret_cast<unsigned long long *>(hist);
    if (threadIdx.x < 3) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) t += wave_sums[w][threadIdx.x];
        if (t != 0.0) atomicAdd(reinterpret_cast<double *>(gc + 5 + NB) + threadIdx.x, t);
    } else if (threadIdx.x >= 64u && threadIdx.x < 64u + 5u) {
        unsigned long long t = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) t += wave_counts[w][threadIdx.x - 64u];
        if (t) atomicAdd(gc + (threadIdx.x - 64u), t);
    } else if (threadIdx.x >= 128u && threadIdx.x < 128u + NB) {
        const uint32_t bin = threadIdx.x - 128u;
        uint32_t t = 0;
#pragma unroll
        for (uint32_t q = 0; q < TILE_COPIES; ++q) t += bins[bin * TILE_COPIES + ((q + bin) & (TILE_COPIES - 1))];
        if (t) atomicAdd(gc + 5 + bin, (unsigned long long)t);
    }
}

mmaemu_status launch_deviation_reset(mmaemu_deviation_hist *h, hipStream_t s)
{
    hipLaunchKernelGGL(deviation_reset_kernel, dim3(1), dim3(128), 0, s, h);
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

constexpr uint64_t TILE_MAX_WORK = 32, TILE_MAX_K = 64;                    // k times the stride; k where every one of many outputs is sampled
constexpr uint64_t TILE_MIN_OUTPUTS = 1ull << 17, TILE_MIN_OUTPUTS_LONG = 1ull << 20;

static mmaemu_status launch_deviation_tiles(const void *A, const void *B, const uint32_t *C, const uint32_t *D, uint32_t m, uint32_t n, uint32_t k,
                                            uint64_t batch, uint32_t ta, uint32_t tb, uint32_t stride, int bin_exp, mmaemu_deviation_hist *h, hipStream_t s)
{
    const bool wide = n % 32 == 0;                             // two blocks of 16 columns per wavefront
    DevTileArgs g = {};
    g.A = (const uint8_t *)A; g.B = (const uint8_t *)B; g.C = C; g.D = D;
    g.m = m; g.n = n; g.k = k; g.ta = ta; g.tb = tb; g.stride = stride; g.bin_exp = bin_exp;
    g.bm = m / 16u; g.bn = n / (wide ? 32u : 16u);
    g.nitems = batch * g.bm * g.bn;
    // An element lies below 2^(E + 1), E its exponent, and is a multiple of 2^(E' - mbits), E' the smallest exponent; k products then
    // reach 2^(E_a + E_b + 2 + ceil(log2 k)) in units of 2^(E'_a + E'_b - mbits_a - mbits_b).
    const FmtInfo fa = fmt_info(ta), fb = fmt_info(tb);
    int lk = 0;
    while ((1u << lk) < k) ++lk;
    g.slack = 53 - 2 - lk - fa.mbits - fb.mbits;
    auto span = [](const FmtInfo &f) { return (1 << f.ebits) - (f.ieee ? 3 : 2); };     // (subnormals are multiples of the smallest normal numbers' unit)
    g.exact_types = span(fa) + span(fb) <= g.slack ? 1u : 0u;
    uint64_t blocks = (g.nitems + 7) / 8;
    const uint64_t most = batch * m * n / stride < 1ull << 40 ? TILE_WORKGROUPS : TILE_WORKGROUPS_MANY;
    if (blocks > most) blocks = most;
    auto go = [&](auto fp8_c) {
        constexpr bool FP8 = decltype(fp8_c)::value;
        if (wide && stride == 1) hipLaunchKernelGGL((deviation_tile_kernel<FP8, 2, false>), dim3((uint32_t)blocks), dim3(512), 0, s, g, h);
        else if (wide) hipLaunchKernelGGL((deviation_tile_kernel<FP8, 2, true>), dim3((uint32_t)blocks), dim3(512), 0, s, g, h);
        else if (stride == 1) hipLaunchKernelGGL((deviation_tile_kernel<FP8, 1, false>), dim3((uint32_t)blocks), dim3(512), 0, s, g, h);
        else hipLaunchKernelGGL((deviation_tile_kernel<FP8, 1, true>), dim3((uint32_t)blocks), dim3(512), 0, s, g, h);
    };
    if (ta == MMAEMU_FP16) go(std::false_type{});
    else go(std::true_type{});
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

// Every stride-th of `total` outputs, output 0 among them (no sum that a large stride could take beyond 64 bits)
static uint64_t samples_of(uint64_t total, uint64_t stride) { return total ? (total - 1) / stride + 1 : 0; }

// The kernel for a call
enum class DevKernel { WholeTiles, FourOutputs, SplitSum, Pairs };

static DevKernel deviation_kernel_for(const void *A, const void *B, const void *C, const void *D, uint32_t m, uint32_t n, uint32_t k, uint64_t batch,
                                      uint32_t ta, uint32_t tb, uint64_t stride)
{
    const uint64_t total = batch * m * n, nsamples = samples_of(total, stride);
    // The split sum for every type but BF16 (whose products span more than the split holds) up to the k for which it is exact.
    // Four outputs of a row per thread where every output is sampled, rows hold whole fours at 16-byte steps, and there are
    // enough of them: a thread then runs four chains, so with few outputs the chip idles behind them, while with many the row of
    // A is decoded once and a quarter of the workgroups end in atomics.  FP16, one / four per thread: 2^12 outputs, k = 1024
    // 91 / 238 us; 2^18, k = 512 81 / 139; 2^19, k = 512 162 / 164; 2^20, k = 512 304 / 264; 2^17, k = 32 14.3 / 14.7;
    // 2^18, k = 32 19.4 / 16.3; 2^19, k = 8 30 / 13.
    const bool split = splits(ta) && splits(tb) && k <= SPLIT_MAX_K;
    const bool fours = split && stride == 1 && n % 4 == 0 && ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(D)) & 15u) == 0;
    const bool wide = fours && (nsamples >= (1ull << 19) || (k <= 32 && nsamples >= (1ull << 18)));
    // Whole tiles on the matrix cores, which form every output's sum whether it is sampled or not and wait for a chunk of k at a time.
    // The other kernels and this one, us, 2^24 outputs of 32x32 FP16 tiles, N(0, 1000): k = 8, strides 1, 2, 3, 5, 8 114, 94, 75, 62, 57 and
    // 47 to 49; k = 16, 32 163, 256 and 54, 89.  Where the exponents lie too far apart (all finite bit patterns, 16x16 tiles):
    // k = 8, 16, 32 at stride 3 87, 109, 142 and 83, 117, 211; at stride 1, 32x32 tiles, k = 8, 32 114, 255 and 82, 202.  2^17
    // outputs of k = 32 17 and 13, 2^14 10 and 11.  Longer rows, stride 1, N(0,1) and finite patterns: 2^24 outputs, k = 40, 64 298, 435 and
    // 111, 188; 298, 438 and 193, 284; 2^20, k = 64 37 and 22, 54 and 31; but 2^17 16 and 20, 25 and 24.
    const bool taken = stride <= TILE_MAX_WORK / k ? total >= TILE_MIN_OUTPUTS : stride == 1 && k <= TILE_MAX_K && total >= TILE_MIN_OUTPUTS_LONG;
    if (((ta == MMAEMU_FP16 && tb == MMAEMU_FP16) || (ta <= MMAEMU_FP8_E5M2 && tb <= MMAEMU_FP8_E5M2)) && m % 16 == 0 && n % 16 == 0 && k % 8 == 0 && taken &&
        n <= (1u << 24) && (uint64_t)m * n <= (1ull << 38) && ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 3u) == 0 &&
        (n % 32 != 0 || ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(D)) & 7u) == 0)) {
        return DevKernel::WholeTiles;
    }
    return wide ? DevKernel::FourOutputs : split ? DevKernel::SplitSum : DevKernel::Pairs;
}

const char *deviation_kernel_name(const void *A, const void *B, const void *C, const void *D, uint32_t m, uint32_t n, uint32_t k, uint64_t batch,
                                  uint32_t ta, uint32_t tb, uint64_t stride)
{
    switch (deviation_kernel_for(A, B, C, D, m, n, k, batch, ta, tb, stride)) {
    case DevKernel::WholeTiles: return "whole tiles";
    case DevKernel::FourOutputs: return "four outputs per thread";
    case DevKernel::SplitSum: return "one output per thread, split sum";
    default: return "one output per thread, pairs";
    }
}

mmaemu_status launch_deviation_sample(const void *A, const void *B, const uint32_t *C, const uint32_t *D, uint32_t m, uint32_t n,
                                      uint32_t k, uint64_t batch, uint32_t ta, uint32_t tb, uint64_t stride, int bin_exp,
                                      mmaemu_deviation_hist *h, hipStream_t s)
{
    const uint64_t nsamples = samples_of(batch * m * n, stride);
    if (nsamples == 0) return MMAEMU_OK;
    if (nsamples > MAX_SAMPLES) { set_error("deviation_sample: more than 2^43 samples in one call"); return MMAEMU_ERR_SHAPE; }
    const DevKernel kernel = deviation_kernel_for(A, B, C, D, m, n, k, batch, ta, tb, stride);
    if (kernel == DevKernel::WholeTiles) return launch_deviation_tiles(A, B, C, D, m, n, k, batch, ta, tb, (uint32_t)stride, bin_exp, h, s);
    const uint64_t nitems = kernel == DevKernel::FourOutputs ? nsamples / 4 : nsamples;
    uint64_t blocks = (nitems + 255) / 256;
    // Grid-stride beyond 2048 workgroups (two rounds of what the chip holds); beyond 2^42 samples 4096, so that no workgroup
    // counts more than 2^31: its rounds of 256 items come to nitems / 2^19 (2^20) rounded up, at most 2^23 rounds of 256 samples
    // or 2^21 of 1024.
    const uint64_t most = nsamples > (1ull << 42) ? 4096 : 2048;
    if (blocks > most) blocks = most;
#define DEVIATION_LAUNCH(W_, S_)                                                                                              \
    hipLaunchKernelGGL((deviation_kernel<W_, S_>), dim3((uint32_t)blocks), dim3(256), 0, s, A, B, C, D, m, n, k, ta, tb, stride, nitems, bin_exp, h)
    if (kernel == DevKernel::FourOutputs) DEVIATION_LAUNCH(4, true);
    else if (kernel == DevKernel::SplitSum) DEVIATION_LAUNCH(1, true);
    else DEVIATION_LAUNCH(1, false);
#undef DEVIATION_LAUNCH
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

} // namespace mmaemu

// Bitwise comparison of two FP32 (or two FP16) outputs with mismatch statistics (paper Eq. 2 and
// Sec. 3.1 Step 4: the model must reproduce the interface bit by bit).
//
// HBM-bound: 8 (4) bytes read per compared pair.  Each lane handles four (eight) consecutive
// elements (one 128-bit load per input), four or two such loads in flight at once; a wavefront whose vectors are equal leaves them alone
// (2^19 equal pairs 6.7 -> 2.3 us, 2^22 7.5 -> 3.4).  The histogram is kept in LDS in 32 copies per
// bucket (copy = lane mod 32), so that lanes counting the same bucket do not serialise
// on one address; counters are flushed with one global atomic per non-zero counter per
// workgroup.
#include "common.hpp"

namespace mmaemu {

__global__ void stats_reset_kernel(mmaemu_stats *st)
{
    uint64_t *w = reinterpret_cast<uint64_t *>(st);
    const uint32_t i = threadIdx.x;
    if (i < sizeof(mmaemu_stats) / 8) w[i] = (i == 3) ? ~0ull : 0ull;   // word 3: first_mismatch_index
}

struct Local {
    uint32_t mism, nan_equiv;
    uint64_t first, maxd;
};

// W = 32: binary32 patterns; W = 16: binary16 patterns (widened to 32 bits by the caller).  The ordered distance of two numbers, the
// difference of their magnitudes' patterns or, across zero, their sum, takes 32 bits (up to twice infinity's pattern, 0xFF000000).
template <int W>
__device__ __forceinline__ void one_pair(uint32_t x, uint32_t y, uint64_t idx, Local &lc, uint32_t &maxd, uint32_t *hist)
{
    constexpr uint32_t SIGN = 1u << (W - 1), MAG = SIGN - 1u, INF = W == 32 ? 0x7F800000u : 0x7C00u;
    const uint32_t ax = x & MAG, ay = y & MAG;
    const bool nx = ax > INF, ny = ay > INF;
    uint32_t bucket;
    if (x != y) {
        lc.first = lc.mism ? lc.first : idx;                         // (a thread's indices ascend)
        lc.mism += 1;
    }
    if (nx || ny) {
        bucket = (nx && ny) ? 0u : 33u;
        if (nx && ny && x != y) lc.nan_equiv += 1;
    } else {
        const uint32_t dist = ((x ^ y) & SIGN) ? ax + ay : max(ax, ay) - min(ax, ay);
        maxd = max(dist, maxd);
        bucket = dist ? 32u - (uint32_t)__builtin_clz(dist) : 0u;
    }
    if (bucket) atomicAdd(&hist[bucket * 32u + (threadIdx.x & 31u)], 1u);   // bucket 0 is derived from the total
}

// the 128 / W elements of one 128-bit load from each input, first element index i0
template <int W>
__device__ __forceinline__ void one_vector(const uint4 &x, const uint4 &y, uint64_t i0, Local &lc, uint32_t &maxd, uint32_t *hist)
{
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (W == 32) {
            one_pair<W>(xs[w], ys[w], i0 + w, lc, maxd, hist);
        } else {
            one_pair<W>(xs[w] & 0xFFFFu, ys[w] & 0xFFFFu, i0 + 2 * w, lc, maxd, hist);
            one_pair<W>(xs[w] >> 16, ys[w] >> 16, i0 + 2 * w + 1, lc, maxd, hist);
        }
    }
}

// (equal vectors count nowhere: a wavefront that meets no other leaves the pairs alone)
__device__ __forceinline__ bool differ(const uint4 &x, const uint4 &y) { return ((x.x ^ y.x) | (x.y ^ y.y) | (x.z ^ y.z) | (x.w ^ y.w)) != 0u; }

// per-workgroup state in LDS
struct WgStats {
    uint32_t hist[34 * 32];
    uint32_t mism, nan_equiv;
    unsigned long long first, maxd;
};

__device__ __forceinline__ void wg_init(WgStats &ws)
{
    for (uint32_t i = threadIdx.x; i < 34 * 32; i += blockDim.x) ws.hist[i] = 0;
    if (threadIdx.x == 0) { ws.mism = 0; ws.nan_equiv = 0; ws.first = ~0ull; ws.maxd = 0; }
    __syncthreads();
}

// lanes -> wavefront -> workgroup -> the caller's struct.  What bounds a comparison beside its bytes is this end: the
// workgroups' atomics meet on the struct's lines.  Nothing is reduced where nothing differs, and all additions of a workgroup
// go out in one instruction (34 lanes folding the histogram, then an atomic per counter one after the other, before): 2^20 pairs,
// equal / 1 % / 80 % differing 8.2 / 12.2 / 12.7 -> 6.9 / 10.6 / 10.7 us; 2^24, 80 % 42.3 -> 33.2 us.
__device__ __forceinline__ void wg_flush(WgStats &ws, Local lc, uint64_t count, mmaemu_stats *st)
{
    unsigned long long *g = reinterpret_cast<unsigned long long *>(st);
    // one set of LDS atomics per wavefront, not per lane: 64 lanes on one address take 64 turns.  Every counter and every
    // bucket but bucket 0 needs a differing pair, so a wavefront without one has nothing to reduce
    if (__ballot(lc.mism != 0u)) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lc.mism += __shfl_xor(lc.mism, o);
            lc.nan_equiv += __shfl_xor(lc.nan_equiv, o);
            const unsigned long long f = __shfl_xor((unsigned long long)lc.first, o), d = __shfl_xor((unsigned long long)lc.maxd, o);
            lc.first = f < lc.first ? f : lc.first;
            lc.maxd = d > lc.maxd ? d : lc.maxd;
        }
        if ((threadIdx.x & 63u) == 0) {
            atomicAdd(&ws.mism, lc.mism);
            atomicMin(&ws.first, (unsigned long long)lc.first);
            if (lc.nan_equiv) atomicAdd(&ws.nan_equiv, lc.nan_equiv);
            if (lc.maxd) atomicMax(&ws.maxd, (unsigned long long)lc.maxd);
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;

    // n_compared and bucket 0 are known up front: workgroup 0 adds the whole count once, every workgroup takes its
    // non-zero buckets back out of bucket 0 (sums are modular, so the order does not matter); equal inputs then cost no
    // further atomics at all
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        atomicAdd(&g[0], (unsigned long long)count);
        atomicAdd(&g[5 + 0], (unsigned long long)count);
    }
    if (!ws.mism) return;
    // The first wavefront folds the histogram, lane = bucket.  The copies are read in rotated order: in plain order all
    // lanes are on one bank in every step.
    uint32_t t = 0;
    if (threadIdx.x >= 1 && threadIdx.x < 34) {
#pragma unroll
        for (uint32_t cpy = 0; cpy < 32; ++cpy) t += ws.hist[threadIdx.x * 32u + ((cpy + threadIdx.x) & 31u)];
    }
    uint32_t nonzero = t;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nonzero += __shfl_xor(nonzero, o);
    // all additions in one instruction, a lane for each word of the struct (the workgroups' atomics meet on its lines)
    unsigned long long add = t;
    uint32_t word = 5u + threadIdx.x;
    if (threadIdx.x == 0) add = 0ull - (unsigned long long)nonzero;
    if (threadIdx.x == 34) { add = ws.mism; word = 1; }
    if (threadIdx.x == 35) { add = ws.nan_equiv; word = 2; }
    if (add) atomicAdd(&g[word], add);
    if (threadIdx.x == 0) {
        atomicMin(&g[3], ws.first);
        if (ws.maxd) atomicMax(&g[4], ws.maxd);
    }
}

// N: 128-bit loads per input in flight
template <int W, int N, typename T>
__global__ void __launch_bounds__(1024)
compare_kernel(const T *__restrict__ d0, const T *__restrict__ d1, uint64_t count, uint64_t base, mmaemu_stats *st)
{
    constexpr uint32_t EPV = 128 / W;                    // elements per 128-bit load
    __shared__ WgStats ws;
    wg_init(ws);
    uint32_t *hist = ws.hist;

    Local lc = {0, 0, ~0ull, 0};
    uint32_t maxd = 0;
    const uint64_t nvec = count / EPV;
    const bool aligned = ((reinterpret_cast<uintptr_t>(d0) | reinterpret_cast<uintptr_t>(d1)) & 15) == 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    if (aligned) {
        const uint4 *v0 = reinterpret_cast<const uint4 *>(d0), *v1 = reinterpret_cast<const uint4 *>(d1);
        uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
        for (; v + (N - 1) * stride < nvec; v += N * stride) {
            uint4 x[N], y[N];
#pragma unroll
            for (int i = 0; i < N; ++i) { x[i] = v0[v + i * stride]; y[i] = v1[v + i * stride]; }
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (__any(differ(x[i], y[i]))) one_vector<W>(x[i], y[i], base + EPV * (v + i * stride), lc, maxd, hist);
        }
        for (; v < nvec; v += stride) {
            const uint4 x = v0[v], y = v1[v];
            if (__any(differ(x, y))) one_vector<W>(x, y, base + EPV * v, lc, maxd, hist);
        }
        for (uint64_t i = EPV * nvec + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
            one_pair<W>(d0[i], d1[i], base + i, lc, maxd, hist);
    } else {
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
            one_pair<W>(d0[i], d1[i], base + i, lc, maxd, hist);
    }
    lc.maxd = maxd;
    wg_flush(ws, lc, count, st);
}

// binary64 patterns: the same statistics; the ordered distance can take 64 bits, and the last distance bucket (32) also
// holds everything from 2^32 upward
__device__ __forceinline__ void one_pair64(uint64_t x, uint64_t y, uint64_t idx, Local &lc, uint32_t *hist)
{
    constexpr uint64_t MAG = 0x7FFFFFFFFFFFFFFFull, INF = 0x7FF0000000000000ull;
    const bool nx = (x & MAG) > INF, ny = (y & MAG) > INF;
    uint32_t bucket;
    if (x != y) {
        lc.mism += 1;
        lc.first = idx < lc.first ? idx : lc.first;
    }
    if (nx || ny) {
        bucket = (nx && ny) ? 0u : 33u;
        if (nx && ny && x != y) lc.nan_equiv += 1;
    } else {
        // |key(x) - key(y)| without leaving 64 bits: same sign: difference of the magnitudes; else their sum (< 2^64)
        const uint64_t ax = x & MAG, ay = y & MAG;
        const uint64_t dist = ((x ^ y) >> 63) ? ax + ay : (ax > ay ? ax - ay : ay - ax);
        lc.maxd = dist > lc.maxd ? dist : lc.maxd;
        const uint32_t bl = dist ? 64u - (uint32_t)__builtin_clzll(dist) : 0u;
        bucket = bl > 32u ? 32u : bl;
    }
    if (bucket) atomicAdd(&hist[bucket * 32u + (threadIdx.x & 31u)], 1u);
}

__global__ void __launch_bounds__(1024)
compare64_kernel(const uint64_t *__restrict__ d0, const uint64_t *__restrict__ d1, uint64_t count, uint64_t base, mmaemu_stats *st)
{
    __shared__ WgStats ws;
    wg_init(ws);
    Local lc = {0, 0, ~0ull, 0};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t nvec = count / 2;
    if (((reinterpret_cast<uintptr_t>(d0) | reinterpret_cast<uintptr_t>(d1)) & 15) == 0) {
        const ulonglong2 *v0 = reinterpret_cast<const ulonglong2 *>(d0), *v1 = reinterpret_cast<const ulonglong2 *>(d1);
        for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvec; v += stride) {
            const ulonglong2 x = v0[v], y = v1[v];
            one_pair64(x.x, y.x, base + 2 * v, lc, ws.hist);
            one_pair64(x.y, y.y, base + 2 * v + 1, lc, ws.hist);
        }
        if ((count & 1) && blockIdx.x == 0 && threadIdx.x == 0) one_pair64(d0[count - 1], d1[count - 1], base + count - 1, lc, ws.hist);
    } else {
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) one_pair64(d0[i], d1[i], base + i, lc, ws.hist);
    }
    wg_flush(ws, lc, count, st);
}

mmaemu_status launch_stats_reset(mmaemu_stats *st, hipStream_t s)
{
    hipLaunchKernelGGL(stats_reset_kernel, dim3(1), dim3(64), 0, s, st);
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

mmaemu_status launch_compare64(const void *d0, const void *d1, uint64_t count, uint64_t base, mmaemu_stats *st, hipStream_t s)
{
    uint64_t blocks = (count + 16383) / 16384;
    blocks = blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks);
    hipLaunchKernelGGL(compare64_kernel, dim3((uint32_t)blocks), dim3(1024), 0, s, (const uint64_t *)d0, (const uint64_t *)d1, count, base, st);
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

// Pairs of binary32 up to which four loads per input are in flight, two beyond: long streams of differing pairs are slower with four.  Two
// and four, us, equal / 0.01 % / 1 % / 80 % differing: 2^22 4.5, 11.4, 15.9, 16.2 and 4.4, 10.8, 16.1, 16.4; 2^24 20.3, 26.6, 28.9, 28.3 and 20.5,
// 26.8, 29.3, 28.5; 2^26 86, 88, 91, 93 and 88, 91, 97, 100; 2^28 345, 346, 357, 357 and 356, 360, 380, 385.  binary16 (twice the arithmetic per
// byte): 2^29 pairs 345, 348, 481, 511 and 358, 365, 468, 496.
constexpr uint64_t COMPARE_FOUR_LOADS = 1ull << 23;

mmaemu_status launch_compare(const void *d0, const void *d1, uint64_t count, uint64_t base, bool half,
                             mmaemu_stats *st, hipStream_t s)
{
    // Few, fat workgroups: a workgroup with differing pairs ends with atomics on up to 38 words of the same few lines, and
    // those serialise across the chip (about 30 ns per workgroup: 2^24 pairs, 256 workgroups, 20.3 us equal and 28.3 differing),
    // so beyond 64 workgroups one covers at least 16K pairs before it pays for them; up to there 4K, one vector of each input per thread (2^14
    // pairs, 80 % differing, workgroups of 4K, 8K, 16K pairs 5.4, 6.3, 8.8 us; 2^18 7.3, 7.1, 9.2; 2^20 14.3, 10.5, 10.9).  1024 threads each, so that a
    // workgroup has 16 waves' worth of loads in flight (a small comparison is latency-bound).  One workgroup per CU at most: with two, equal inputs streamed
    // 4 % faster, but inputs that differ paid twice the atomics (15 % more at 2^24 pairs, measured when each counter was an
    // atomic of its own), and the closed-loop workloads compare mostly differing outputs.
    const uint64_t fine = (count + 4095) / 4096, fat = (count + 16383) / 16384;
    uint64_t blocks = fine < 64 ? fine : (fat > 64 ? fat : 64);
    if (blocks < 1) blocks = 1;
    if (blocks > 256) blocks = 256;
    if (half)
        hipLaunchKernelGGL((compare_kernel<16, 4, uint16_t>), dim3((uint32_t)blocks), dim3(1024), 0, s, (const uint16_t *)d0,
                           (const uint16_t *)d1, count, base, st);
    else if (count <= COMPARE_FOUR_LOADS)
        hipLaunchKernelGGL((compare_kernel<32, 4, uint32_t>), dim3((uint32_t)blocks), dim3(1024), 0, s, (const uint32_t *)d0,
                           (const uint32_t *)d1, count, base, st);
    else
        hipLaunchKernelGGL((compare_kernel<32, 2, uint32_t>), dim3((uint32_t)blocks), dim3(1024), 0, s, (const uint32_t *)d0,
                           (const uint32_t *)d1, count, base, st);
    MMAEMU_HIP(hipGetLastError());
    return MMAEMU_OK;
}

} // namespace mmaemu

// The closed-loop scan in one launch (Sec. 3.1 Step 4: many candidate parameter sets over the same random tiles, each
// compared bit by bit with a reference, Eq. 2): up to MULTI_MAX models of one family and of *any* group length, internal
// width and fold period share the staged operands of a pass.  Families (one kernel instantiation each): T-FDPA with the
// accumulator inside the sum; TR-FDPA (the accumulator added after the products' sum, with the two round-downs and the
// variation switches); TR-FDPA on groups split in halves or quarters; GTR-FDPA (the even / odd split).  What follows
// describes the first; the others differ in what a group's maximum covers and in the group epilogue.
//
// Staging and decoding A and B, loading C and the reference and forming the exponent maxima cost about as much as
// running one model, so that part is paid once per pass for all the models of a launch:
//   * a workgroup pass stages four 16x16x16 or 16x16x32 tiles (one 32x32x8 or 32x32x16 tile), the whole k at once, as the
//     single-model kernels of emulate_tiled.hpp do (same LDS layout and helpers);
//   * pass 1 runs once at the finest granularity, a quarter group of four products: the packed 16-bit maximum of each
//     quarter is kept in LDS, two quarters per dword and thread;
//   * the model loop reads per model six scalars from the kernel-argument segment (F, switches, output mask, NaN
//     pattern, L, arithmetic kind); a group's maximum is the maximum of its quarters; pass 2 is a run-time loop over
//     the group in steps of four k (one 128-bit LDS read per row and step);
//   * arithmetic kinds: 0, the whole group summed in 32 bits; 1, folded into binary64 every four terms; 2, every term;
//     3, F of 30 and more: terms truncated and summed in binary64 (values widened on load where the chunk is held in
//     binary32);
//   * group epilogue: the binary64 route of the single-model kernels, or (kind 0, every output of the wavefront with a
//     normal result and no tagged element) a 32-bit route: the accumulator aligned like a product, the sum an integer,
//     rho one int -> float conversion under the wavefront's rounding mode and an exact scaling;
//   * every output is compared with the reference in registers; a differing output does one LDS atomic on a histogram
//     bucket, the largest distance and first index are reduced over the wavefront by row shifts; a persistent workgroup
//     writes its non-zero counters out once, at its end (a global atomic on a shared cache line costs about as much as a
//     thousand instructions of a wave).
// Models that flush subnormal inputs come last in a launch (the staged values are flushed in place once).
//
// T-FDPA on tiles of up to 16 k (FAST) goes further.  The kernel is bound by vector-ALU issue, and of the 10.7 (FP8) to 11.5
// (BF16) instructions per term that the loop above took, the products (formed again for every model from LDS: 1 of 4 in pass
// 2, and in binary64 for BF16, where the LDS reads were as long as the arithmetic), the group ends and the statistics were
// what many models can share or a shorter form can do:
//   * a thread's four outputs keep all their products in registers (64 for 16 k), formed once per pass (and once more where
//     models flush their inputs); BF16 products are held in binary32 relative to their quarter's maximum exponent;
//   * groups are unrolled, exponents stay biased, the scale's inverse takes the place of a second scaling: 13 instead of 24
//     instructions per group end; the kept maxima, the accumulators and the reference outputs wait in LDS as 128-bit words;
//   * special values follow from one IEEE sum per group, taken only by wavefronts that hold any (bit patterns full of NaNs
//     ran at half the speed of ordinary data through the routes of the general loop);
//   * the reference's ordered keys are formed once per pass, a histogram entry is counted by leading zeros, and the two
//     reductions over the wavefront run only where they can change something.
// Launches of six and more TR-FDPA sets on all operands but BF16 go the same way (FAM 4): the sixteen sets of the closed-loop scan
// on 2^15 tiles of 16x16x16 FP16, N(0,1) operands, 566 -> 523 us.  At four waves per SIMD 15 registers of a thread lie in scratch memory on
// 16x16x16, 8 on 32x32x16 and none on 32x32x8.  Three waves and four, us: six and sixteen sets on
// 2^15 tiles of 16x16x16 252, 542 and 241, 501, 2^13 of 32x32x16 239, 536 and 227, 495, of 32x32x8 186, 376 and 148, 330; but 2^12 tiles of
// 16x16x16 59, 107 and 75, 119, 2^9 25, 52 and 26, 53.
// Measured (kernel times), one launch of the sixteen sets of the closed-loop scan on 2^16 tiles of 16x16x16, before and after: FP8 1108 ->
// 670 us (6.22 instructions per term), BF16 bit patterns 1433 -> 1137 us (8.70), all FP16 bit patterns (a quarter of the
// tiles) 571 -> 253 us; three sets on 2^18 tiles of 32x32x8 1953 -> 1354 us (7.31).  What is left is still issue: 0.84 to
// 1.02 of the nominal rate, one instruction per SIMD in four cycles, which is no ceiling: independent v_mul_f32 and v_add_u32, half of a
// term's instructions, issue at 1.4 to 1.6 of it, the others at 0.82 to 0.93.
#include "emulate_tiled.hpp"
#include <atomic>

namespace mmaemu {

struct ScanArgs {
    uint32_t ta, tb;
    int32_t ebase;                     // Exp = e' + ebase for a product
    uint32_t count;                    // models in this launch, 1 .. MULTI_MAX
    uint32_t ref_is_first;             // no reference array: the first model's outputs are the reference
    const uint32_t *dref;              // reference outputs [batch][m][n], or null
    uint32_t *dout;                    // null, or every model's outputs: model i at dout + slot[i] * out_stride
    uint64_t out_stride, index_base;
    uint64_t *stats;                   // the caller's mmaemu_stats array as 64-bit words
    uint32_t zbias;                    // ZBIAS when zero terms stay out of the exponent maxima (TR-FDPA sets with that switch), else 0
    uint32_t slot[MULTI_MAX];
    struct Hot { int32_t F; uint32_t flags, out_mask, nan_bits, L, kind; int32_t F2, Fc, drop, Fm; uint32_t parts, twin; } hot[MULTI_MAX];
};

__device__ __forceinline__ ScanArgs::Hot scan_hot(uint32_t mi)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) ScanArgs *KArgs;
    KArgs sa = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
    ScanArgs::Hot h;
    h.F = sa->hot[mi].F; h.flags = sa->hot[mi].flags; h.out_mask = sa->hot[mi].out_mask; h.nan_bits = sa->hot[mi].nan_bits;
    h.L = sa->hot[mi].L; h.kind = sa->hot[mi].kind;
    h.F2 = sa->hot[mi].F2; h.Fc = sa->hot[mi].Fc; h.drop = sa->hot[mi].drop; h.Fm = sa->hot[mi].Fm; h.parts = sa->hot[mi].parts; h.twin = sa->hot[mi].twin;
    return h;
#else
    return ScanArgs::Hot{};
#endif
}

// TM x TM x KC tiles (16 x 16 x 16, 16 x 16 x 32, 32 x 32 x 8 or 32 x 32 x 16: the whole k of a tile is staged at once), 2 x 2
// outputs per thread; ADAPT: BF16 operands, whose staged chunk is
// held in binary64 when any element lies outside [2^-31, 2^32).
// (Four waves per SIMD are asked for outright where the LDS allows four workgroups per CU: left alone the compiler settles
// at about 150 vector registers and three waves; the handful of registers that go to scratch instead cost less than the
// fourth wave brings: +6 %.  Five waves were slower.  The BF16 kernels that keep 64 products take three: they hold about 140
// registers, and 16 x 16 x 16's LDS holds three workgroups.  The 16 x 16 x 32 instantiations hold two or three
// workgroups per CU and are compiled for that many waves.)
// A kept quarter maximum (FAM 0: biased exponent) at or above this one holds a NaN or an infinity.
constexpr uint32_t TAGGED = 0x2000u;

__device__ __forceinline__ uint32_t opaque_thread_index()
{
    uint32_t t = threadIdx.x;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(t));
#endif
    return t;
}

// Ordered key of a binary32 pattern that is no NaN (sign-magnitude patterns read as integers: -|x| for a negative x, x
// for a positive one), plus 2^31; |key(x) - key(y)| is then one v_sad_u32 (the compiler makes none of these by itself).
__device__ __forceinline__ uint32_t ordered_key(uint32_t x)
{
    const uint32_t s = (uint32_t)((int32_t)x >> 31);                       // 0 or all ones
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t c, k;
    asm("v_bfi_b32 %0, %1, 1, %2" : "=v"(c) : "v"(s), "s"(0x80000000u));   // s ? 1 : 2^31
    asm("v_xad_u32 %0, %1, %2, %3" : "=v"(k) : "v"(x), "v"(s), "v"(c));    // (x ^ s) + c
    return k;
#else
    return (x ^ s) + (s ? 1u : 0x80000000u);
#endif
}
__device__ __forceinline__ uint32_t key_distance(uint32_t kx, uint32_t ky)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t d;
    asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(kx), "v"(ky));
    return d;
#else
    return kx > ky ? kx - ky : ky - kx;
#endif
}
// A value that every lane of the wavefront holds alike, in a scalar register.
__device__ __forceinline__ uint32_t scalar(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// The products of a thread's outputs fit its registers: T-FDPA, and TR-FDPA on binary32 values, on tiles of up to 16 k.
template <int KC, int FAM> constexpr bool scan_fast() { return FAM == 4 || (FAM == 0 && KC <= 16); }

// LDS of one workgroup: staged values and exponents, the kept quarter maxima, the statistics
template <int TM, int KC, bool ADAPT, int FAM>
constexpr int scan_lds_bytes()
{
    constexpr int SLOTS = 256 / ((TM / 2) * (TM / 2));
    constexpr int VS = KC + 4, VSD = KC + 2, ES = KC / 2 + (KC == 8 ? 4 : 2);
    constexpr int KEPT = FAM == 3 ? KC / 4 : (KC / 4 + 1) / 2;            // dwords of kept maxima per output
    return 2 * SLOTS * TM * (ADAPT ? VSD * 8 : VS * 4) + 2 * SLOTS * TM * ES * 4 + KEPT * 4 * 256 * 4 + (scan_fast<KC, FAM>() ? 3 : 0) * 4 * 256 * 4 +
           (int)sizeof(MultiLds) + 16;
}
// workgroups (of four waves, one per SIMD) that a CU's 160 KB of LDS hold, four at most: the waves per SIMD to compile for
template <int TM, int KC, bool ADAPT, int FAM>
constexpr int scan_waves()
{
    constexpr int by_lds = (160 * 1024) / scan_lds_bytes<TM, KC, ADAPT, FAM>();
    constexpr int most = FAM == 0 && KC == 16 && ADAPT ? 3 : 4;
    return by_lds >= most ? most : by_lds;
}

// FAM 0: T-FDPA, the accumulator a term of the sum; FAM 1: TR-FDPA (unsplit groups), the accumulator added after the
// products' sum with the two round-downs; FAM 2: GTR-FDPA's merge of sub-group sums with the sub-groups being the two
// halves or the four quarters of a group (binary32 values only: FP8 / FP16 operands, a sub-group's sum in 32 bits); FAM 3:
// GTR-FDPA as printed, the sub-groups being the even and the odd products; FAM 4: FAM 1 on binary32 values (all operands but BF16) and
// up to 16 k, with the products in registers.
// TWIN (FAM 0, tiles of one group): a model marked `twin` is followed by one that differs from it only in the output
// conversion (rounding, E8M13, output flush, NaN pattern); the two share the group's maximum and sum, and only the end of
// the group and the statistics run twice.
template <int TM, int KC, bool ADAPT, int FAM, bool TWIN>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(scan_waves<TM, KC, ADAPT, FAM>(), scan_waves<TM, KC, ADAPT, FAM>())))
emulate_scan_kernel(ScanArgs sa_, const void *__restrict__ A, const void *__restrict__ B, const uint32_t *Cm, uint64_t nitems, uint32_t nblocks)
{
    constexpr int R = 2, C = 2, TN = TM;
    constexpr int TI = TM / R, TJ = TN / C, TPS = TI * TJ, SLOTS = 256 / TPS;
    static_assert(TPS * SLOTS == 256, "thread layout");
    constexpr bool FAST = scan_fast<KC, FAM>();
    constexpr int VS = KC + 4, VSD = KC + 2, ES = KC / 2 + (KC == 8 ? 4 : 2);
    constexpr int NQ4 = KC / 4;                                   // quarter groups per row
    constexpr int NK2 = (NQ4 + 1) / 2;                            // dwords of kept maxima per output
    constexpr int VBYTES = SLOTS * TM * (ADAPT ? VSD * 8 : VS * 4);
    constexpr int EBYTES = SLOTS * TM * ES * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * VBYTES + 2 * EBYTES];
    // (one 128-bit LDS word holds a kept dword of all four outputs of a thread; FAM 3: a quarter's even and odd maximum, one dword)
    __shared__ __attribute__((aligned(16))) uint32_t m2k[FAM == 3 ? NQ4 : NK2][256][R * C];
    // (FAST: the accumulators, the reference outputs and their keys wait in LDS, not in registers that the products need)
    __shared__ __attribute__((aligned(16))) uint32_t c0_kept[FAST ? 256 : 1][R * C], ref_kept[FAST ? 256 : 1][R * C], ref_key[FAST ? 256 : 1][R * C];
    __shared__ MultiLds ml;
    constexpr int HC = HIST_COPIES;
    uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < MULTI_MAX * 34 * HC; i += 256) (&ml.hist[0][0][0])[i] = 0;
    if (tid < MULTI_MAX) { ml.naneq[tid] = 0; ml.maxd[tid] = 0; ml.first[tid] = ~0ull; }
    // (FAST, ADAPT) some element of the pass needs binary64 products: a flag by the pass's parity, set before a barrier, read
    // after it and cleared after the next pass's: one barrier instead of a reduction's three
    __shared__ volatile uint32_t flag_wild[2];
    uint32_t parity = 0;
    if constexpr (FAST && ADAPT) {
        if (tid < 2) flag_wild[tid] = 0u;
        __syncthreads();
    }
    // (the first staging's barriers come before any thread counts anything)

    unsigned char *Av_raw = smem, *Bv_raw = smem + VBYTES;
    uint32_t *Ae = reinterpret_cast<uint32_t *>(smem + 2 * VBYTES);
    uint32_t *Be = reinterpret_cast<uint32_t *>(smem + 2 * VBYTES + EBYTES);
    const ScanArgs *sa = reinterpret_cast<const ScanArgs *>(opaque_kernarg_ptr());
    uint32_t slot = tid / TPS, ti = (tid % TPS) / TJ, tj = tid % TJ;
    const uint32_t ta = sa_.ta, tb = sa_.tb;
    const int ebase = sa_.ebase;
    const uint32_t esa = (ta <= MMAEMU_FP8_E5M2 || ta >= MMAEMU_FP6_E2M3) ? 1u : 2u;
    const uint32_t esb = (tb <= MMAEMU_FP8_E5M2 || tb >= MMAEMU_FP6_E2M3) ? 1u : 2u;
    const float *av, *bv;
    const double *avd, *bvd;
    const uint32_t *ae, *be;
    auto find_rows = [&] {
        av = reinterpret_cast<const float *>(Av_raw) + (slot * TM + ti) * VS;
        bv = reinterpret_cast<const float *>(Bv_raw) + (slot * TN + tj) * VS;
        avd = reinterpret_cast<const double *>(Av_raw) + (slot * TM + ti) * VSD;
        bvd = reinterpret_cast<const double *>(Bv_raw) + (slot * TN + tj) * VSD;
        ae = Ae + (slot * TM + ti) * ES;
        be = Be + (slot * TN + tj) * ES;
    };
    find_rows();
    // AGAIN (64 products in four waves' registers): a thread's places are worked out again for every pass and every forming of the
    // products; kept across the models they sent 8 to 12 registers to scratch memory, 2 to 4 % of a launch of one set
    constexpr bool AGAIN = FAST && KC == 16 && !ADAPT;
    auto places_again = [&] {
        if constexpr (AGAIN) {
            tid = opaque_thread_index();
            slot = TPS == 256 ? 0u : tid / TPS;
            ti = (tid % TPS) / TJ;
            tj = tid % TJ;
            find_rows();
        }
    };
    const uint32_t count = sa_.count, ref_first = sa_.ref_is_first;
    uint32_t found = 0;                        // models for which this wavefront has put a first differing index into LDS
    const bool dumping = sa_.dout != nullptr;
    const uint32_t *dref = sa->dref;

    // Staging: the tiles of a pass lie one after the other and are staged whole, so quad q of a panel (four consecutive k of
    // one row) starts 4 q elements behind the pass's first element: one scalar base and a 32-bit offset per thread.  Where
    // both panels together have at most 256 quads (32 x 32 tiles) a wavefront stages one of A's or one of B's, not both.
    constexpr int QUADS = SLOTS * TM * (KC / 4);
    constexpr bool SHARED_PASS = 2 * QUADS <= 256;
    constexpr int NQ = SHARED_PASS ? 1 : (QUADS + 255) / 256;
    constexpr int NM = SHARED_PASS ? 1 : 2;                      // panels a thread has a hand in
    static_assert(SHARED_PASS ? (QUADS % 64 == 0 && 256 % QUADS == 0) : QUADS % 256 == 0, "quads per thread");
    const bool stages_b = SHARED_PASS && (__builtin_amdgcn_readfirstlane((int)tid) / QUADS) % 2 != 0;      // (uniform over a wavefront)
    auto quad_of = [&](int i) -> uint32_t { return SHARED_PASS ? tid % QUADS : tid + 256u * i; };
    auto load_quads = [&](const void *base, uint32_t es, uint64_t first_item, uint2 (&raw)[NQ]) {
        const uint64_t left = nitems - first_item;               // (surplus slots of the last pass re-read its last tile)
        const uint8_t *p0 = static_cast<const uint8_t *>(base) + first_item * (uint64_t)(TM * KC) * es;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const uint32_t q = quad_of(i), sl = q / (TM * KC / 4);
            uint32_t e = 4u * q;
            if (left < SLOTS && sl >= (uint32_t)left) e -= (sl - ((uint32_t)left - 1u)) * (uint32_t)(TM * KC);
            if (es == 1) { raw[i].x = *reinterpret_cast<const uint32_t *>(p0 + e); raw[i].y = 0; }
            else raw[i] = *reinterpret_cast<const uint2 *>(p0 + 2u * e);
        }
    };
    auto load_pass = [&](uint64_t first_item, uint2 (&raw)[NM][NQ]) {
        if constexpr (SHARED_PASS) load_quads(stages_b ? B : A, stages_b ? esb : esa, first_item, raw[0]);
        else {
            load_quads(A, esa, first_item, raw[0]);
            load_quads(B, esb, first_item, raw[NM - 1]);
        }
    };
    auto store_quads = [&](bool is_b, const float (&f)[NQ][4], const uint2 (&x)[NQ], bool as_double) {
        unsigned char *const lv = is_b ? Bv_raw : Av_raw;
        uint32_t *const le = is_b ? Be : Ae;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const uint32_t q = quad_of(i), row = q / (KC / 4), kq = q % (KC / 4);
            *reinterpret_cast<uint2 *>(le + row * ES + 2 * kq) = x[i];
            if (as_double) {
                double *dst = reinterpret_cast<double *>(lv) + row * VSD + 4 * kq;
                *reinterpret_cast<double2 *>(dst) = make_double2((double)f[i][0], (double)f[i][1]);
                *reinterpret_cast<double2 *>(dst + 2) = make_double2((double)f[i][2], (double)f[i][3]);
            } else {
                *reinterpret_cast<float4 *>(reinterpret_cast<float *>(lv) + row * VS + 4 * kq) = make_float4(f[i][0], f[i][1], f[i][2], f[i][3]);
            }
        }
    };
    // first output of the thread, counted from the pass's first (surplus slots: the last tile's)
    auto out_offset = [&](uint64_t first_item) -> uint32_t {
        const uint64_t left = nitems - first_item;
        const uint32_t sl = (left < SLOTS && slot >= (uint32_t)left) ? (uint32_t)left - 1u : slot;
        return (sl * TM + ti) * TN + tj;                         // + TI * r * TN + TJ * c
    };
    // AHEAD (the 32 x 32 tiles of FP8 / FP16 operands, whose kernels have registers to spare under the four-wave budget):
    // a pass's global loads (operand quads, accumulator inputs, reference) are issued one pass ahead, right after the
    // previous pass has been staged, so that they arrive while its models run.
    constexpr bool AHEAD = TM == 32 && !ADAPT && FAM == 0;
    constexpr int NA = AHEAD ? NQ : 1, RA = AHEAD ? R : 1, CA = AHEAD ? C : 1;
    uint2 nraw[NM][NA];
    uint32_t nc0[RA][CA], nref[RA][CA];
    auto fetch_pass = [&](uint32_t wg) {
        if constexpr (AHEAD) {
            const uint64_t it0 = (uint64_t)wg * SLOTS;
            load_pass(it0, nraw);
            const uint32_t off = out_offset(it0);
            const uint32_t *cp = Cm + it0 * (uint64_t)(TM * TN), *rp = dref + it0 * (uint64_t)(TM * TN);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    nc0[r][c] = cp[off + (TI * r) * TN + TJ * c];
                    nref[r][c] = ref_first ? 0u : rp[off + (TI * r) * TN + TJ * c];
                }
        }
    };
    if (AHEAD && blockIdx.x < nblocks) fetch_pass(blockIdx.x);
    for (uint32_t pass_wg = blockIdx.x; pass_wg < nblocks; pass_wg += gridDim.x) {
        places_again();
        // ---- this pass's tiles: outputs, operands in flight ----
        const uint64_t item0 = (uint64_t)pass_wg * SLOTS;
        const uint64_t out0 = item0 * (uint64_t)(TM * TN);
        uint2 raw[NM][NQ];
        if constexpr (AHEAD) {
#pragma unroll
            for (int w = 0; w < NM; ++w)
#pragma unroll
                for (int q = 0; q < NQ; ++q) raw[w][q] = nraw[w][q];
        } else {
            load_pass(item0, raw);
        }
        const bool live = scalar(item0 + slot < nitems ? 1u : 0u) != 0;      // (a wavefront works on one tile)
        const uint32_t d_off = out_offset(item0);                // (behind out0)
        uint32_t c0[R][C], ref[R][C];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if constexpr (AHEAD) {
                    c0[r][c] = nc0[r][c];
                    ref[r][c] = nref[r][c];
                } else {
                    const uint32_t o = d_off + (TI * r) * TN + TJ * c;
                    c0[r][c] = (Cm + out0)[o];
                    ref[r][c] = ref_first ? 0u : (dref + out0)[o];
                }
            }
        // ---- decode and stage (as the first model wants them) ----
        bool chunk_is_double = false;
        int staged;
        {
            const uint32_t ftz0 = scan_hot(0).flags & FL_FTZ_IN;
            staged = ftz0 ? 1 : 0;
            float f[NM][NQ][4];
            uint2 x[NM][NQ];
            const uint32_t zbias = FAM != 0 ? sa_.zbias : 0u;
            bool wild = decode_any<NQ>(stages_b ? tb : ta, raw[0], ftz0, zbias, f[0], x[0]);
            if constexpr (NM == 2) wild |= decode_any<NQ>(tb, raw[1], ftz0, zbias, f[1], x[1]);
            // (the barrier also protects the previous pass's readers)
            if constexpr (ADAPT && FAST) {
                if (wild) flag_wild[parity] = 1u;
                __syncthreads();
                chunk_is_double = __builtin_amdgcn_readfirstlane((int)flag_wild[parity]) != 0;
                if (tid == 0) flag_wild[parity ^ 1u] = 0u;
                parity ^= 1u;
            } else if (ADAPT) chunk_is_double = __syncthreads_or(wild) != 0;
            else __syncthreads();
            store_quads(stages_b, f[0], x[0], chunk_is_double);
            if constexpr (NM == 2) store_quads(true, f[1], x[1], chunk_is_double);
            __syncthreads();
        }
        if (AHEAD && pass_wg + gridDim.x < nblocks) fetch_pass(pass_wg + gridDim.x);
        // ---- pass 1, once: the maximum of e'_a + e'_b over each quarter group, two quarters per kept dword ----
        uint32_t top = 0;                                         // (FAST) the largest kept maximum of the thread's outputs
#pragma unroll
        for (int q = 0; q < NQ4; ++q) {
            uint2 ea[R], eb[C];
#pragma unroll
            for (int r = 0; r < R; ++r) ea[r] = *reinterpret_cast<const uint2 *>(ae + TI * r * ES + 2 * q);
#pragma unroll
            for (int c = 0; c < C; ++c) eb[c] = *reinterpret_cast<const uint2 *>(be + TJ * c * ES + 2 * q);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const uint32_t x = pk_max_u16(pk_add_u16(ea[r].x, eb[c].x), pk_add_u16(ea[r].y, eb[c].y));
                    const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                    uint32_t mx = lo > hi ? lo : hi;
                    if constexpr (FAM == 0) {
                        // kept as a biased binary32 exponent, 1 at least (the accumulator's own is never below 1, so what lies
                        // under it cannot be the group's maximum); a tagged one stays far above every other
                        const int mb = (int)mx + ebase + 127;
                        mx = mb < 1 ? 1u : (uint32_t)mb;
                    }
                    if constexpr (FAST) top = mx > top ? mx : top;
                    // (each thread its own words: no barrier needed)
                    if constexpr (FAM == 3) m2k[q][tid][r * C + c] = x;           // low half: the even k, high half: the odd k
                    else if (q % 2 == 0) m2k[q / 2][tid][r * C + c] = mx;
                    else m2k[q / 2][tid][r * C + c] |= mx << 16;
                }
        }

        // ---- a model's outputs against the reference ----
        // Per output that differs: one LDS atomic on its histogram bucket (bucket 0 of the LDS copy counts pairs that
        // differ at distance 0: zeros of both signs, NaNs of two patterns), so the number of mismatches is the
        // histogram's sum.  The largest distance is reduced over the wavefront only where it passes the one in LDS, and
        // the first index once per wavefront and model: a workgroup's passes go through ascending tiles, so no later
        // pass can lower it.
        // (An LDS histogram is kept by leading zeros of the distance: place 32 - bucket, and 33 for bucket 33.  FAST: the keys of
        // the reference outputs sit in LDS, formed once per pass; the other families, with fewer models to share them, form a key
        // where it is needed.)
        uint32_t ref_nan = 1u;                                    // some reference output of the wavefront may be a NaN
        auto take_reference = [&](const uint32_t (&ref)[R][C]) {
            bool any = false;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    any |= (ref[r][c] & 0x7FFFFFFFu) > 0x7F800000u;
                    if (FAST) {
                        ref_key[tid][r * C + c] = ordered_key(ref[r][c]);
                        ref_kept[tid][r * C + c] = ref[r][c];
                    }
                }
            ref_nan = scalar(__any(any) ? 1u : 0u);
        };
        if (!ref_first) take_reference(ref);
        // every NaN becomes the model's pattern; returns whether the wavefront holds one
        auto write_nan = [&](uint32_t (&x)[R][C], uint32_t nan_pattern) -> bool {
            bool any = false;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if ((x[r][c] & 0x7FFFFFFFu) > 0x7F800000u) {
                        x[r][c] = nan_pattern;
                        any = true;
                    }
            return scalar(__any(any) ? 1u : 0u) != 0u;
        };
        // (x: the model's outputs, every NaN already the model's pattern; nan_seen: there may be one)
        auto account = [&](uint32_t mi, const uint32_t (&x)[R][C], bool nan_seen) {
            if (!live) return;
            const uint32_t tid = opaque_thread_index();           // (addresses formed here, not kept across the models' loop)
            uint32_t *dout = nullptr;
            uint64_t dump_off = 0;
            if (dumping) { dout = sa->dout; dump_off = (uint64_t)sa->slot[mi] * sa->out_stride + out0; }       // (uniform)
            uint32_t maxd = 0;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (dumping) (dout + dump_off)[d_off + (TI * r) * TN + TJ * c] = x[r][c];
                }
            if (__builtin_expect(ref_first && mi == 0, 0)) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) ref[r][c] = x[r][c];
                take_reference(x);
                return;                                           // (its own row reports no mismatch)
            }
            uint32_t y[R][C];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) y[r][c] = FAST ? ref_kept[tid][r * C + c] : ref[r][c];
            uint32_t *const hist = &ml.hist[mi][0][tid & (HC - 1)];
            if (__builtin_expect(nan_seen || ref_nan != 0u, 0)) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        if (x[r][c] != y[r][c]) {
                            const uint32_t dist = key_distance(ordered_key(x[r][c]), FAST ? ref_key[tid][r * C + c] : ordered_key(y[r][c]));
                            const bool nx = (x[r][c] & 0x7FFFFFFFu) > 0x7F800000u, ny = (y[r][c] & 0x7FFFFFFFu) > 0x7F800000u;
                            uint32_t place = (uint32_t)__clz((int)dist);                                  // (__clz(0) = 32)
                            if (nx || ny) {
                                place = (nx && ny) ? 32u : 33u;
                                if (nx && ny) atomicAdd(&ml.naneq[mi], 1u);                               // (rare)
                            } else {
                                maxd = dist > maxd ? dist : maxd;
                            }
                            atomicAdd(hist + place * HC, 1u);
                        }
                    }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (x[r][c] != y[r][c]) {
                            const uint32_t dist = key_distance(ordered_key(x[r][c]), FAST ? ref_key[tid][r * C + c] : ordered_key(y[r][c]));
                            maxd = dist > maxd ? dist : maxd;
                            atomicAdd(hist + (uint32_t)__clz((int)dist) * HC, 1u);
                        }
            }
            if (scalar(__any(maxd > ml.maxd[mi]) ? 1u : 0u)) {
                const uint32_t wmax = wave_reduce_to_lane63<true>(maxd);
                if ((tid & 63u) == 63u) atomicMax(&ml.maxd[mi], wmax);
            }
            if (!((found >> mi) & 1u)) {
                uint32_t rel = 0xFFFFFFFFu;
#pragma unroll
                for (int r = R - 1; r >= 0; --r)
#pragma unroll
                    for (int c = C - 1; c >= 0; --c)
                        if (x[r][c] != y[r][c]) rel = d_off + (uint32_t)((TI * r) * TN + TJ * c);
                if (scalar(__any(rel != 0xFFFFFFFFu) ? 1u : 0u)) {
                    const uint32_t wmin = wave_reduce_to_lane63<false>(rel);
                    if ((tid & 63u) == 63u) atomicMin(&ml.first[mi], (unsigned long long)(sa->index_base + out0 + wmin));
                    found |= 1u << mi;
                }
                found = scalar(found);
            }
        };

        if constexpr (FAST) {
            // ---- the products of the thread's outputs in registers, shared by all the models ----
            // special: an operand of the wavefront's is a NaN or an infinity, or an accumulator is one or may become one.  The
            // groups' results then follow Sec. 4.2 through an IEEE sum of the group's products and its accumulator (special_sum).
            // (An infinity that a BF16 chain reaches by overflow is no such case: it stays by itself, see rho32.)
            bool odd = top >= (FAM == 0 ? TAGGED : SENTINEL);
            // TR-FDPA's last steps keep an infinite or NaN accumulator by themselves, so only operands ask for that sum: six and twelve sets on
            // 2^15 tiles of 16x16x16, N(0,1) operands and all accumulators, 287, 479 us with it and 273, 446 without
            const bool special_operand = FAM == 4 && scalar(__any(odd) ? 1u : 0u) != 0u;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    c0_kept[tid][r * C + c] = c0[r][c];
                    odd |= ((c0[r][c] >> 23) & 0xFFu) >= 254u;      // (FP8 / FP16 sums stay below 2^40: from 253 no chain overflows)
                }
            const bool special = scalar(__any(odd) ? 1u : 0u) != 0u;
            {
                // (the scheduler would interleave the outputs' sums and the quarters' products, for registers that go to scratch memory)
                auto one_at_a_time = [] {
#if defined(__HIP_DEVICE_COMPILE__)
                    __builtin_amdgcn_sched_barrier(0);
#endif
                };
                float p[R][C][KC];
                auto kept = [&](int q, int r, int c) -> uint32_t { return (m2k[q / 2][tid][r * C + c] >> (16 * (q & 1))) & 0xFFFFu; };
                // p = a b, exact; BF16: a b 2^-(quarter's maximum exponent), exact wherever the term can reach the sum's unit
                // (a product 2^-126 below its quarter's largest is cut to zero at any width).  In a quarter with a NaN or an
                // infinity the finite products are scaled away.
                auto form_products = [&](bool flush) {
                    places_again();
                    const float min_a = flush ? min_normal_of(ta) : 0.0f, min_b = flush ? min_normal_of(tb) : 0.0f;
#pragma unroll
                    for (int q = 0; q < NQ4; ++q) {
                        int down[ADAPT ? R : 1][ADAPT ? C : 1];          // the power of two that a quarter's products are scaled by
                        if constexpr (ADAPT) {
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) down[r][c] = 127 - (int)kept(q, r, c);
                            if (__builtin_expect(special, 0)) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) down[r][c] = down[r][c] < -400 ? -400 : down[r][c];
                            }
                        }
                        if (ADAPT && chunk_is_double) {
                            double sc[ADAPT ? R : 1][ADAPT ? C : 1];
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) if constexpr (ADAPT) sc[r][c] = __hiloint2double((1023 + down[r][c]) << 20, 0);
#pragma unroll
                            for (int h = 0; h < 4; h += 2) {
                                double a[R][2], b[C][2];
#pragma unroll
                                for (int r = 0; r < R; ++r) {
                                    const double2 v = *reinterpret_cast<const double2 *>(avd + TI * r * VSD + 4 * q + h);
                                    a[r][0] = __builtin_fabs(v.x) < (double)min_a ? 0.0 : v.x;
                                    a[r][1] = __builtin_fabs(v.y) < (double)min_a ? 0.0 : v.y;
                                }
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    const double2 v = *reinterpret_cast<const double2 *>(bvd + TJ * c * VSD + 4 * q + h);
                                    b[c][0] = __builtin_fabs(v.x) < (double)min_b ? 0.0 : v.x;
                                    b[c][1] = __builtin_fabs(v.y) < (double)min_b ? 0.0 : v.y;
                                }
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        p[r][c][4 * q + h] = (float)((a[r][0] * b[c][0]) * sc[ADAPT ? r : 0][ADAPT ? c : 0]);
                                        p[r][c][4 * q + h + 1] = (float)((a[r][1] * b[c][1]) * sc[ADAPT ? r : 0][ADAPT ? c : 0]);
                                    }
                            }
                            one_at_a_time();
                        } else {
                            float a[R][4], b[C][4];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const float4 v = *reinterpret_cast<const float4 *>(av + TI * r * VS + 4 * q);
                                a[r][0] = v.x; a[r][1] = v.y; a[r][2] = v.z; a[r][3] = v.w;
                            }
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const float4 v = *reinterpret_cast<const float4 *>(bv + TJ * c * VS + 4 * q);
                                b[c][0] = v.x; b[c][1] = v.y; b[c][2] = v.z; b[c][3] = v.w;
                            }
                            if (flush) {
#pragma unroll
                                for (int w = 0; w < 4; ++w) {
#pragma unroll
                                    for (int r = 0; r < R; ++r) a[r][w] = __builtin_fabsf(a[r][w]) < min_a ? 0.0f : a[r][w];
#pragma unroll
                                    for (int c = 0; c < C; ++c) b[c][w] = __builtin_fabsf(b[c][w]) < min_b ? 0.0f : b[c][w];
                                }
                            }
#pragma unroll
                            for (int w = 0; w < 4; ++w)
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        const float x = a[r][w] * b[c][w];
                                        p[r][c][4 * q + w] = ADAPT ? ldexpf(x, down[ADAPT ? r : 0][ADAPT ? c : 0]) : x;
                                    }
                            one_at_a_time();
                        }
                    }
                };
                form_products(false);
                bool flushed = staged != 0;
#pragma unroll 1
                for (uint32_t mi = 0; mi < count; ++mi) {
                    const ScanArgs::Hot hot = scan_hot(mi);
                    const int F = hot.F;
                    const uint32_t fl = hot.flags;
                    const bool twin = TWIN && hot.twin != 0;
                    if ((fl & FL_FTZ_IN) && !flushed) { form_products(true); flushed = true; }
                    if constexpr (FAM == 0) set_f32_round_toward_zero((fl & FL_RZ) != 0);
                    // (the kept maxima are read again for every model: hoisted out of this loop they would take up to 28 registers)
                    const uint32_t tid = opaque_thread_index();
                    auto kept = [&](int q, int r, int c) -> uint32_t { return (m2k[q / 2][tid][r * C + c] >> (16 * (q & 1))) & 0xFFFFu; };
                    uint32_t d[R][C], d2[R][C] = {};
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) d[r][c] = c0_kept[tid][r * C + c];
                    // rho of a 32-bit sum S in units of 2^(emb - 127 - F): one int -> float conversion under the wavefront's
                    // rounding mode, then an exact scaling; the result is zero or normal
                    auto rho32 = [&](int32_t S, float back, uint32_t emb, uint32_t dp, uint32_t fe, uint32_t om) -> uint32_t {
                        const float f = (float)S;
                        uint32_t o;
                        if constexpr (ADAPT) {
                            o = __float_as_uint(ldexpf(f, (int)emb - (F + 127)));
                            if (fe & FL_RZ) {
                                if ((o & 0x7FFFFFFFu) == 0x7F800000u) o -= 1u;             // overflow: the largest finite number
                                o &= om;
                            }
                            if ((dp & 0x7F800000u) == 0x7F800000u) o = dp;                 // an infinity that the chain has reached stays
                        } else {
                            o = __float_as_uint(f * back);
                            if (fe & FL_RZ) o &= om;
                        }
                        return o;
                    };
                    auto rho64 = [&](double v, uint32_t fe, uint32_t om) -> uint32_t {
                        uint32_t o = __float_as_uint((float)v);
                        if (fe & FL_RZ) {
                            const double b = (double)__uint_as_float(o);
                            if (__builtin_fabs(b) > __builtin_fabs(v)) o -= 1u;            // rounded away from zero: step back
                            o &= om;
                        }
                        if (ADAPT && (fe & FL_FTZ_OUT) && (o & 0x7F800000u) == 0) o &= 0x80000000u;
                        return o;
                    };
                    // rho of a 32-bit sum whose result may be subnormal
                    auto rho_low = [&](int32_t S, uint32_t emb, uint32_t dp, uint32_t fe, uint32_t om) -> uint32_t {
                        const uint32_t o = rho64(ldexp((double)S, (int)emb - (F + 127)), fe, om);
                        return (dp & 0x7F800000u) == 0x7F800000u ? dp : o;                     // (as in rho32)
                    };
                    // Sec. 4.2 for group g of GL products: their IEEE sum with the accumulator is a NaN or an infinity exactly where
                    // the group's result is (finite products are far too small to make one), and is then that result; the
                    // infinities that BF16 chains reach by overflow stay through it too.
                    auto special_sum = [&](auto gl_c, int g, int r, int c, uint32_t dp) -> uint32_t {
                        constexpr int GL = decltype(gl_c)::value;
                        float t = p[r][c][g * GL];
#pragma unroll
                        for (int w = 1; w < GL; ++w) t += p[r][c][g * GL + w];
                        return __float_as_uint(t + __uint_as_float(dp));
                    };
                    auto run_fast = [&](auto gl_c, auto wide_c) {
                        constexpr int GL = decltype(gl_c)::value;
                        constexpr bool WIDE = decltype(wide_c)::value != 0, PAIRS = decltype(wide_c)::value == 1;
                        if constexpr (GL <= KC) {
#pragma unroll
                        for (int g = 0; g < KC / GL; ++g) {
                            uint32_t emb[R][C], before[R][C];      // the group's maximum exponent, biased; its accumulator
                            bool low = false;
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    uint32_t e;
                                    if constexpr (GL == 4) e = kept(g, r, c);
                                    else {
                                        uint32_t x = m2k[g * (GL / 8)][tid][r * C + c];
#pragma unroll
                                        for (int i = 1; i < GL / 8; ++i) x = pk_max_u16(x, m2k[g * (GL / 8) + i][tid][r * C + c]);
                                        const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                                        e = lo > hi ? lo : hi;
                                    }
                                    const uint32_t Ec = (d[r][c] >> 23) & 0xFFu;
                                    emb[r][c] = e > Ec ? e : Ec;
                                    if constexpr (ADAPT && !WIDE) low |= emb[r][c] < (uint32_t)(F + 1);
                                }
                            // (a group of the wavefront's whose result may be subnormal: its 32-bit sums are converted from binary64)
                            const bool some_low = ADAPT && !WIDE && __any(low);
                            if constexpr (!WIDE) {
                                if (ADAPT && some_low && (fl & FL_FTZ_IN)) {
#pragma unroll
                                    for (int r = 0; r < R; ++r)
#pragma unroll
                                        for (int c = 0; c < C; ++c) if ((d[r][c] & 0x7F800000u) == 0) d[r][c] = 0;      // FlushSubnormal on the accumulator
                                }
                                int32_t S[R][C];
                                float back[R][C];
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        float scale;
                                        if constexpr (ADAPT) {
                                            // (the accumulator's exponent may lie anywhere below the group's maximum)
                                            S[r][c] = (int32_t)ldexpf(__uint_as_float(d[r][c]), (F + 127) - (int)emb[r][c]);
                                            back[r][c] = 0.0f;
                                        } else {
                                            const uint32_t sb = (uint32_t)(F + 254 - (int)emb[r][c]) << 23;         // 2^(F - e_max), normal
                                            scale = __uint_as_float(sb);
                                            back[r][c] = __uint_as_float(0x7F000000u - sb);                        // its inverse
                                            S[r][c] = (int32_t)(__uint_as_float(d[r][c]) * scale);
                                        }
#pragma unroll
                                        for (int q = 0; q < GL / 4; ++q) {
                                            if constexpr (ADAPT) {
                                                const int se = (F + 127) + (int)kept(g * (GL / 4) + q, r, c) - (int)emb[r][c];
                                                scale = __uint_as_float((uint32_t)(se < 1 ? 1 : se) << 23);
                                            }
#pragma unroll
                                            for (int w = 0; w < 4; ++w) S[r][c] += (int32_t)(p[r][c][g * GL + 4 * q + w] * scale);
                                        }
                                        one_at_a_time();
                                    }
                                if constexpr (TWIN && GL == KC) {
                                    if (twin) {
                                        const ScanArgs::Hot h2 = scan_hot(mi + 1);
                                        set_f32_round_toward_zero((h2.flags & FL_RZ) != 0);
                                        auto second = [&](auto low_c) {
#pragma unroll
                                            for (int r = 0; r < R; ++r)
#pragma unroll
                                                for (int c = 0; c < C; ++c) {
                                                    // (a copy the optimiser cannot see through: to it the conversions under the two rounding modes are one)
                                                    int32_t S2 = S[r][c];
#if defined(__HIP_DEVICE_COMPILE__)
                                                    asm volatile("" : "+v"(S2));
#endif
                                                    if constexpr (decltype(low_c)::value) d2[r][c] = rho_low(S2, emb[r][c], d[r][c], h2.flags, h2.out_mask);
                                                    else d2[r][c] = rho32(S2, back[r][c], emb[r][c], d[r][c], h2.flags, h2.out_mask);
                                                }
                                        };
                                        if (ADAPT && __builtin_expect(some_low, 0)) second(std::true_type{}); else second(std::false_type{});
                                        set_f32_round_toward_zero((fl & FL_RZ) != 0);
                                    }
                                }
                                auto first = [&](auto low_c) {
#pragma unroll
                                    for (int r = 0; r < R; ++r)
#pragma unroll
                                        for (int c = 0; c < C; ++c) {
                                            before[r][c] = d[r][c];
                                            if constexpr (decltype(low_c)::value) d[r][c] = rho_low(S[r][c], emb[r][c], d[r][c], fl, hot.out_mask);
                                            else d[r][c] = rho32(S[r][c], back[r][c], emb[r][c], d[r][c], fl, hot.out_mask);
                                        }
                                };
                                if (ADAPT && __builtin_expect(some_low, 0)) first(std::true_type{}); else first(std::false_type{});
                            } else {
                                double v[R][C];
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        // (FlushSubnormal on the accumulator, and on the result below: FP8 / FP16 products keep
                                        // every group's unit far above the subnormals, whose aligned image is zero)
                                        if (ADAPT && (fl & FL_FTZ_IN) && (d[r][c] & 0x7F800000u) == 0) d[r][c] = 0;
                                        const int unit = (int)emb[r][c] - 127 - F;
                                        double T = 0.0 + __builtin_trunc(ldexp((double)__uint_as_float(d[r][c]), -unit));      // (+0.0 whatever the signs)
                                        float scale = __uint_as_float((uint32_t)(F + 254 - (int)emb[r][c]) << 23);
#pragma unroll
                                        for (int q = 0; q < GL / 4; ++q) {
                                            if constexpr (ADAPT) {
                                                const int se = (F + 127) + (int)kept(g * (GL / 4) + q, r, c) - (int)emb[r][c];
                                                scale = __uint_as_float((uint32_t)(se < 1 ? 1 : se) << 23);
                                            }
                                            // aligned and truncated in binary32, exactly; PAIRS: two terms to a 32-bit sum
#pragma unroll
                                            for (int w = 0; w < 4; w += 2) {
                                                const float t0 = p[r][c][g * GL + 4 * q + w] * scale, t1 = p[r][c][g * GL + 4 * q + w + 1] * scale;
                                                if constexpr (PAIRS) T += (double)((int32_t)t0 + (int32_t)t1);
                                                else {
                                                    T += (double)__builtin_truncf(t0);
                                                    T += (double)__builtin_truncf(t1);
                                                }
                                            }
                                        }
                                        v[r][c] = ldexp(T, unit);                                                  // exact: integers below 2^53
                                        one_at_a_time();
                                    }
                                if constexpr (TWIN && GL == KC) {
                                    if (twin) {
                                        // (the binary64 -> binary32 conversion follows the binary32 rounding mode too)
                                        const ScanArgs::Hot h2 = scan_hot(mi + 1);
                                        set_f32_round_toward_zero((h2.flags & FL_RZ) != 0);
#pragma unroll
                                        for (int r = 0; r < R; ++r)
#pragma unroll
                                            for (int c = 0; c < C; ++c) {
                                                double v2 = v[r][c];
#if defined(__HIP_DEVICE_COMPILE__)
                                                asm volatile("" : "+v"(v2));                   // (as for S2 above)
#endif
                                                d2[r][c] = rho64(v2, h2.flags, h2.out_mask);
                                            }
                                        set_f32_round_toward_zero((fl & FL_RZ) != 0);
                                    }
                                }
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        before[r][c] = d[r][c];
                                        d[r][c] = rho64(v[r][c], fl, hot.out_mask);
                                    }
                            }
                            if (__builtin_expect(special, 0)) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        const uint32_t t = special_sum(gl_c, g, r, c, before[r][c]);
                                        const bool sp = (t & 0x7F800000u) == 0x7F800000u;
                                        d[r][c] = sp ? t : d[r][c];
                                        if (TWIN && GL == KC) d2[r][c] = sp ? t : d2[r][c];
                                        one_at_a_time();
                                    }
                            }
                        }
                        }
                    };
                    // TR-FDPA: the products' sum alone at their own maximum exponent, then the last steps of all four outputs side by side.
                    // WIDTH 0: the group's aligned terms in 32 bits; 1: two terms to a 32-bit sum, the sums in binary64; 2: one by one.
                    auto run_rd = [&](auto gl_c, auto width_c) {
                        constexpr int GL = decltype(gl_c)::value, WIDTH = decltype(width_c)::value;
                        if constexpr (GL <= KC && FAM == 4) {
#pragma unroll
                        for (int g = 0; g < KC / GL; ++g) {
                            double T[R * C], v[R * C];
                            int em[R * C];
                            uint32_t cb[R * C], o[R * C];
                            bool have[R * C];
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    const int i = r * C + c;
                                    uint32_t e;
                                    if constexpr (GL == 4) e = kept(g, r, c);
                                    else {
                                        uint32_t x = m2k[g * (GL / 8)][tid][i];
#pragma unroll
                                        for (int j = 1; j < GL / 8; ++j) x = pk_max_u16(x, m2k[g * (GL / 8) + j][tid][i]);
                                        const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                                        e = lo > hi ? lo : hi;
                                    }
                                    em[i] = (int)e + ebase;
                                    have[i] = !(fl & FL_SKIP_ZERO) || e >= 2 * ZBIAS;
                                    cb[i] = d[r][c];
                                    int se = F + 127 - em[i];
                                    se = se < 1 ? 1 : (se > 254 ? 254 : se);                       // (the clamps never change a truncated term)
                                    const float scale = __uint_as_float((uint32_t)se << 23);
                                    if constexpr (WIDTH == 0) {
                                        int32_t S = 0;
#pragma unroll
                                        for (int w = 0; w < GL; ++w) S += (int32_t)(p[r][c][g * GL + w] * scale);
                                        T[i] = (double)S;
                                    } else {
                                        T[i] = 0.0;
#pragma unroll
                                        for (int w = 0; w < GL; w += 2) {
                                            const float t0 = p[r][c][g * GL + w] * scale, t1 = p[r][c][g * GL + w + 1] * scale;
                                            if constexpr (WIDTH == 1) T[i] += (double)((int32_t)t0 + (int32_t)t1);
                                            else {
                                                T[i] += (double)__builtin_truncf(t0);
                                                T[i] += (double)__builtin_truncf(t1);
                                            }
                                        }
                                    }
                                    one_at_a_time();
                                }
                            if (fl & FL_FTZ_IN) {
#pragma unroll
                                for (int i = 0; i < R * C; ++i) if ((cb[i] & 0x7F800000u) == 0) cb[i] = 0;             // FlushSubnormal on the accumulator
                            }
                            bool low = true;                          // some result may be a zero of negative sign
                            if (__builtin_expect((fl & FL_SUM_EXACT) != 0u, 1)) low = rd_exact_all<false>(T, em, F, cb, hot.F2, hot.Fc, hot.drop, fl, v);
                            else {
#pragma unroll
                                for (int i = 0; i < R * C; ++i) v[i] = rd_general(T[i], have[i], em[i], F, cb[i], hot.F2, hot.Fc, hot.drop, fl);
                            }
#pragma unroll
                            for (int i = 0; i < R * C; ++i) o[i] = __float_as_uint((float)v[i]);
                            if ((fl & (FL_RZ | FL_FTZ_OUT)) != 0u || (low && (fl & FL_ZERO_POSITIVE) != 0u)) {         // (one test on the common way)
#pragma unroll
                                for (int i = 0; i < R * C; ++i) {
                                    if (fl & FL_RZ) {
                                        const double back = (double)__uint_as_float(o[i]);
                                        if (__builtin_fabs(back) > __builtin_fabs(v[i])) o[i] -= 1u;               // rounded away from zero: step back
                                        o[i] &= hot.out_mask;                                                      // RZ-E8M13 cuts further, still toward zero
                                    }
                                    if ((fl & FL_FTZ_OUT) && (o[i] & 0x7F800000u) == 0) o[i] &= 0x80000000u;
                                    if ((fl & FL_ZERO_POSITIVE) && (o[i] & 0x7FFFFFFFu) == 0) o[i] = 0u;
                                }
                            }
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    if (__builtin_expect(special_operand, 0)) {
                                        const uint32_t t = special_sum(gl_c, g, r, c, d[r][c]);
                                        if ((t & 0x7F800000u) == 0x7F800000u) o[r * C + c] = t;
                                        one_at_a_time();
                                    }
                                    d[r][c] = o[r * C + c];
                                }
                        }
                        }
                    };
                    auto by_width = [&](auto gl_c) {
                        constexpr int GL = decltype(gl_c)::value;
                        if constexpr (FAM == 4) {
                            if (hot.kind == 0) run_rd(gl_c, std::integral_constant<int, 0>{});
                            else if (F <= 28) run_rd(gl_c, std::integral_constant<int, 1>{});
                            else run_rd(gl_c, std::integral_constant<int, 2>{});
                            return;
                        }
                        const bool fits = F >= 1 && F <= 28 && ((uint64_t)(GL + 1) << (F + 2)) <= (1ull << 31);
                        if (fits) { run_fast(gl_c, std::integral_constant<int, 0>{}); return; }
                        // (an aligned term is below 2^(F+2): two of them stay inside 32 bits up to F = 28)
                        const bool pairs = (2ull << (F + 2)) <= (1ull << 31);
                        if (pairs) run_fast(gl_c, std::integral_constant<int, 1>{}); else run_fast(gl_c, std::integral_constant<int, 2>{});
                    };
                    if (hot.L == 4) by_width(std::integral_constant<int, 4>{});
                    else if (hot.L == 8) by_width(std::integral_constant<int, 8>{});
                    else by_width(std::integral_constant<int, 16>{});
                    if (__builtin_expect(special, 0)) write_nan(d, hot.nan_bits);
                    account(mi, d, special);
                    if (twin) {
                        ++mi;
                        if (__builtin_expect(special, 0)) write_nan(d2, scan_hot(mi).nan_bits);
                        account(mi, d2, special);
                    }
                }
                set_f32_round_toward_zero(false);
            }
        } else {
        // ---- the models ----
        {
#pragma unroll 1
        for (uint32_t mi = 0; mi < count; ++mi) {
            const ScanArgs::Hot hot = scan_hot(mi);
            const int F = hot.F;
            const uint32_t fl = hot.flags, L = hot.L, kind = hot.kind;
            typename std::conditional<TWIN, uint32_t, const uint32_t>::type out_mask = hot.out_mask, nan_bits = hot.nan_bits;
            typename std::conditional<TWIN, uint32_t, const uint32_t>::type fe = fl;   // the switches the end of a group reads (a twin brings its own)
            const bool twin = TWIN && hot.twin != 0;
            uint32_t dfirst[R][C];                            // the first model's outputs of a pair of twins
            const uint32_t nan_first = hot.nan_bits;
            (void)kind;
            if ((fl & FL_FTZ_IN) && !staged) {
                // FlushSubnormal on the staged values, in place (exponents do not change: a subnormal keeps Exp = 1 - bias)
                __syncthreads();
                const float min_a = min_normal_of(ta), min_b = min_normal_of(tb);
                if (chunk_is_double) {
                    double *va = reinterpret_cast<double *>(Av_raw), *vb = reinterpret_cast<double *>(Bv_raw);
                    _Pragma("unroll 1") for (uint32_t i = tid; i < SLOTS * TM * VSD; i += 256) if (__builtin_fabs(va[i]) < (double)min_a) va[i] = 0.0;
                    _Pragma("unroll 1") for (uint32_t i = tid; i < SLOTS * TN * VSD; i += 256) if (__builtin_fabs(vb[i]) < (double)min_b) vb[i] = 0.0;
                } else {
                    float *va = reinterpret_cast<float *>(Av_raw), *vb = reinterpret_cast<float *>(Bv_raw);
                    _Pragma("unroll 1") for (uint32_t i = tid; i < SLOTS * TM * VS; i += 256) if (__builtin_fabsf(va[i]) < min_a) va[i] = 0.0f;
                    _Pragma("unroll 1") for (uint32_t i = tid; i < SLOTS * TN * VS; i += 256) if (__builtin_fabsf(vb[i]) < min_b) vb[i] = 0.0f;
                }
                __syncthreads();
                staged = 1;
            }
            // rho = RZ-FP32: the short route's int -> float conversion truncates under the binary32 rounding mode "toward
            // zero" (every other binary32 operation of the loop is exact in either mode, and the binary64 route checks the
            // direction of its own conversion)
            if constexpr (FAM == 0) set_f32_round_toward_zero((fl & FL_RZ) != 0);
            uint32_t d[R][C];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < C; ++c) d[r][c] = c0[r][c];
            bool slow_seen = false;                           // some group left the short route (a NaN may have come out of it)
            // (families with round-downs) the output conversions other than round to nearest, from the exact values
            auto convert_rare = [&](const double (&v)[R][C], uint32_t (&dn)[R][C]) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        uint32_t o = dn[r][c];
                        if ((fl & FL_RZ)) {
                            const double back = (double)__uint_as_float(o);
                            if (__builtin_fabs(back) > __builtin_fabs(v[r][c])) o -= 1u;       // rounded away from zero: step back
                            o &= out_mask;                                                     // RZ-E8M13 cuts further, still toward zero
                        }
                        if ((fl & FL_FTZ_OUT) && (o & 0x7F800000u) == 0) o &= 0x80000000u;
                        if ((fl & FL_ZERO_POSITIVE) && (o & 0x7FFFFFFFu) == 0) o = 0u;
                        dn[r][c] = o;
                    }
            };
            // The groups of one model, specialised on the group length GL and the arithmetic kind so that the loops
            // unroll and the LDS addresses of a group are immediate offsets.
            auto run_groups = [&](auto gl_c, auto kind_c) {
                constexpr int GL = decltype(gl_c)::value, KIND = decltype(kind_c)::value;
                constexpr int U2 = (GL / 4 <= 2) ? 2 : 1;             // (a whole group of 16 in flight costs a wave of occupancy)
                if constexpr (GL <= KC && FAM <= 1) {
                const bool fits = KIND == 0 && ((uint64_t)(GL + 1) << (F + 2)) <= (1ull << 31) && F >= 1;
#pragma unroll 1
                for (int g = 0; g < KC / GL; ++g) {
                    const uint32_t kg = g * GL;
                    // e_max of the group: its quarters' maxima, then the accumulator
                    int emax[R][C];
                    uint32_t tagged = 0, tg[R][C];
                    bool have[R][C];                          // (FAM 1) a product took part
                    auto group_max = [&](int r, int c) -> uint32_t {
                        if constexpr (GL == 4) {
                            return (m2k[g / 2][tid][r * C + c] >> (16 * (g & 1))) & 0xFFFFu;
                        } else {
                            uint32_t x = m2k[g * (GL / 8)][tid][r * C + c];
#pragma unroll
                            for (int i = 1; i < GL / 8; ++i) x = pk_max_u16(x, m2k[g * (GL / 8) + i][tid][r * C + c]);
                            const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                            return lo > hi ? lo : hi;
                        }
                    };
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            uint32_t e = group_max(r, c);
                            const int em = FAM == 0 ? (int)e - 127 : (int)e + ebase;
                            have[r][c] = true;
                            if constexpr (FAM == 1) {
                                // (zero terms kept out of the maxima: a product with a zero factor has an exponent sum below 2 ZBIAS)
                                have[r][c] = !(fl & FL_SKIP_ZERO) || e >= 2 * ZBIAS;
                                // a BF16 product may reach 2^128, which this family counts as an infinity: tagged, and settled
                                // from the staged values (such a chunk is held in binary64, where products are exact)
                                if (ADAPT && em >= 127 && !(e & 0xC000u)) e |= 0x8000u;
                                tg[r][c] = e & 0xC000u;
                                tagged |= e;
                                emax[r][c] = em;
                                continue;
                            }
                            tg[r][c] = e >= TAGGED ? 0xC000u : 0u;
                            tagged |= tg[r][c];
                            uint32_t dd = d[r][c];
                            if ((fl & FL_FTZ_IN) && (dd & 0x7F800000u) == 0) { dd = 0; d[r][c] = 0; }     // FlushSubnormal on the accumulator
                            const uint32_t Ec = (dd >> 23) & 0xFFu;                                        // (a flushed subnormal keeps Exp = -126)
                            const int ec = (int)(Ec ? Ec : 1u) - 127;
                            emax[r][c] = ec > em ? ec : em;
                        }
                    tagged &= 0xC000u;
                    // ---- pass 2 ----
                    int32_t S32[R][C];
                    double Sd[R][C];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) { S32[r][c] = 0; Sd[r][c] = 0.0; }
                    auto fold = [&]() {
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) { Sd[r][c] += (double)S32[r][c]; S32[r][c] = 0; }
                    };
                    float fscale[R][C];                           // 2^(F - e_max) in binary32, where pass 2 runs in binary32
                    if ((ADAPT && chunk_is_double) || KIND == 3) {
                        // binary64: exact product, exact scaling; the float -> int conversion truncates, or (KIND 3: F of 30
                        // and more) v_trunc_f64 and a binary64 sum, exact below 2^53
                        double scale[R][C];
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) scale[r][c] = __hiloint2double((F - emax[r][c] + 1023) << 20, 0);   // 2^(F - e_max), always normal
#pragma unroll 1
                        for (int q = 0; q < GL; q += 2) {
                            double a[R][2], b[C][2];
                            if (ADAPT && chunk_is_double) {
#pragma unroll
                                for (int r = 0; r < R; ++r) { const double2 v = *reinterpret_cast<const double2 *>(avd + TI * r * VSD + kg + q); a[r][0] = v.x; a[r][1] = v.y; }
#pragma unroll
                                for (int c = 0; c < C; ++c) { const double2 v = *reinterpret_cast<const double2 *>(bvd + TJ * c * VSD + kg + q); b[c][0] = v.x; b[c][1] = v.y; }
                            } else {
#pragma unroll
                                for (int r = 0; r < R; ++r) { const float2 v = *reinterpret_cast<const float2 *>(av + TI * r * VS + kg + q); a[r][0] = (double)v.x; a[r][1] = (double)v.y; }
#pragma unroll
                                for (int c = 0; c < C; ++c) { const float2 v = *reinterpret_cast<const float2 *>(bv + TJ * c * VS + kg + q); b[c][0] = (double)v.x; b[c][1] = (double)v.y; }
                            }
#pragma unroll
                            for (int w = 0; w < 2; ++w) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        const double t = (a[r][w] * b[c][w]) * scale[r][c];
                                        if constexpr (KIND == 3) Sd[r][c] += __builtin_trunc(t);
                                        else S32[r][c] += (int32_t)t;
                                    }
                                if constexpr (KIND == 2) fold();
                            }
                            if constexpr (KIND == 1) { if ((q & 2) != 0) fold(); }
                        }
                    } else {
                        // binary32 values: the product is exact, the scaling aligns it, the conversion truncates toward zero
                        float (&scale)[R][C] = fscale;
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                int se = F + 127 - emax[r][c];                         // biased exponent of 2^(F - e_max)
                                se = se < 1 ? 1 : (se > 254 ? 254 : se);               // the clamps never change a truncated term
                                scale[r][c] = __uint_as_float((uint32_t)se << 23);
                            }
#pragma unroll U2
                        for (int q = 0; q < GL; q += 4) {
                            float a[R][4], b[C][4];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const float4 v = *reinterpret_cast<const float4 *>(av + TI * r * VS + kg + q);
                                a[r][0] = v.x; a[r][1] = v.y; a[r][2] = v.z; a[r][3] = v.w;
                            }
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const float4 v = *reinterpret_cast<const float4 *>(bv + TJ * c * VS + kg + q);
                                b[c][0] = v.x; b[c][1] = v.y; b[c][2] = v.z; b[c][3] = v.w;
                            }
#pragma unroll
                            for (int w = 0; w < 4; ++w) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) S32[r][c] += (int32_t)((a[r][w] * b[c][w]) * scale[r][c]);
                                if constexpr (KIND == 2) fold();
                            }
                            if constexpr (KIND == 1) fold();
                        }
                    }

                    // ---- end of the group ----
                    // Short route: when the GL truncated products and the truncated accumulator together fit 32 bits, the
                    // accumulator is aligned like a product, the whole sum is a 32-bit integer, and rho is the int -> float
                    // conversion followed by an exact scaling -- as long as the result cannot be subnormal and nothing is
                    // tagged: e_max - F >= -126 and e_max <= 127 for every output of the wavefront.
                    uint32_t dkeep[TWIN ? R : 1][TWIN ? C : 1];
                    if constexpr (TWIN) {
                        if (twin) {
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) dkeep[r][c] = d[r][c];
                        }
                    }
                    constexpr int TWINS = TWIN ? 2 : 1;
#pragma unroll 1
                    for (int tw = 0; tw < TWINS && (tw == 0 || twin); ++tw) {
                    if constexpr (TWIN) {
                        if (tw == 1) {
                            // the twin: the first model's outputs aside, the accumulator back, the twin's output conversion
                            const ScanArgs::Hot h2 = scan_hot(mi + 1);
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) { dfirst[r][c] = d[r][c]; d[r][c] = dkeep[r][c]; }
                            if constexpr (TWIN) {
                                fe = h2.flags;
                                out_mask = h2.out_mask;
                                nan_bits = h2.nan_bits;
                            }
                            set_f32_round_toward_zero((fe & FL_RZ) != 0);
                        }
                    }
                    bool done = false;
                    if constexpr (KIND == 0 && FAM == 0) {
                        if (fits) {
                            uint32_t worst = tagged ? 0xFFFFFFFFu : 0u;
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    const uint32_t u = (uint32_t)(emax[r][c] - (F - 126));          // 0 .. 253 - F on this route
                                    worst = u > worst ? u : worst;
                                }
                            if (__all(worst <= (uint32_t)(253 - F))) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) {
                                        // 2^(F - e_max), a normal number on this route (so pass 2's clamps left it alone)
                                        // (the BF16 kernels form it again: kept across their binary64 branch it costs registers)
                                        const float scale = ADAPT ? __uint_as_float((uint32_t)(F + 127 - emax[r][c]) << 23) : fscale[r][c];
                                        const int32_t S = S32[r][c] + (int32_t)(__uint_as_float(d[r][c]) * scale);
                                        const float f = (float)S;                                  // (truncates under RZ)
                                        uint32_t o = __float_as_uint(ldexpf(f, emax[r][c] - F));
                                        if ((fe & FL_RZ)) {
                                            if ((o & 0x7FFFFFFFu) == 0x7F800000u) o -= 1u;         // overflow: the largest finite number
                                            o &= out_mask;
                                        }
                                        d[r][c] = o;
                                    }
                                done = true;
                            }
                        }
                    }
                    if (!done) {
                        slow_seen = true;
                        uint32_t dn[R][C];
                        double vrd[R][C];                         // (FAM 1) the value to convert; one branch on the way for all four outputs
                        bool low = true;                          // (FAM 1) some result may be a zero of negative sign
                        if constexpr (FAM == 1) {
                            if (fl & FL_FTZ_IN) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) if ((d[r][c] & 0x7F800000u) == 0) d[r][c] = 0;             // FlushSubnormal on the accumulator
                            }
                            auto sum = [&](int r, int c) -> double { return KIND == 0 ? (double)S32[r][c] : Sd[r][c] + (double)S32[r][c]; };
                            if (__builtin_expect((fl & FL_SUM_EXACT) != 0u, 0)) {
                                const double T[4] = {sum(0, 0), sum(0, 1), sum(1, 0), sum(1, 1)};
                                const int em[4] = {emax[0][0], emax[0][1], emax[1][0], emax[1][1]};
                                const uint32_t cb[4] = {d[0][0], d[0][1], d[1][0], d[1][1]};
                                double v[4];
                                low = rd_exact_all<false>(T, em, F, cb, hot.F2, hot.Fc, hot.drop, fl, v);
                                vrd[0][0] = v[0]; vrd[0][1] = v[1]; vrd[1][0] = v[2]; vrd[1][1] = v[3];
                            } else {
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) vrd[r][c] = rd_general(sum(r, c), have[r][c], emax[r][c], F, d[r][c], hot.F2, hot.Fc, hot.drop, fl);
                            }
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const double T = Sd[r][c] + (double)S32[r][c];
                                double v;
                                if constexpr (FAM == 0) {
                                    const int unit = emax[r][c] - F;
                                    // the accumulator, aligned and truncated like every other term
                                    const double tc = __builtin_trunc(ldexp((double)__uint_as_float(d[r][c]), -unit));
                                    v = ldexp(T + tc, unit);                                   // exact: integers below 2^53
                                } else {
                                    v = vrd[r][c];
                                }
                                uint32_t o = __float_as_uint((float)v);
                                if (FAM == 0 && (fe & FL_RZ)) {
                                    const double back = (double)__uint_as_float(o);
                                    if (__builtin_fabs(back) > __builtin_fabs(v)) o -= 1u;     // rounded away from zero: step back
                                    o &= out_mask;                                             // RZ-E8M13 cuts further, still toward zero
                                }
                                if (FAM == 0 && (fe & FL_FTZ_OUT) && (o & 0x7F800000u) == 0) o &= 0x80000000u;
                                dn[r][c] = o;
                            }
                        if constexpr (FAM == 1) {
                            // (one test on the common way)
                            if ((fl & (FL_RZ | FL_FTZ_OUT)) != 0u || (low && (fl & FL_ZERO_POSITIVE) != 0u)) convert_rare(vrd, dn);
                        }
                        if (tagged) {
                            // NaN and infinite operands (Sec. 4.2): classes and signs from the staged values
                            const bool dbl = ADAPT && chunk_is_double;
                            const void *pa = dbl ? static_cast<const void *>(avd + kg) : static_cast<const void *>(av + kg);
                            const void *pb = dbl ? static_cast<const void *>(bvd + kg) : static_cast<const void *>(bv + kg);
                            // (FAM 1: under the product-overflow rule a finite product of 2^128 or more counts as an infinity;
                            // a group tagged for its large maximum alone in which no product gets there keeps the value above)
                            const uint2 sp = special_products<R, C, TI * VS, TJ * VS, TI * VSD, TJ * VSD, GL>(pa, pb, (dbl ? 1u : 0u) | (FAM == 1 ? 2u : 0u));
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c)
                                    if (tg[r][c]) {
                                        const uint32_t i = r * C + c, cb = d[r][c];
                                        bool nn = (sp.x >> i) & 1u, pp = (sp.y >> i) & 1u, mm = (sp.y >> (16 + i)) & 1u;
                                        if ((cb & 0x7FFFFFFFu) > 0x7F800000u) nn = true;                       // the accumulator joins
                                        else if ((cb & 0x7FFFFFFFu) == 0x7F800000u) { if (cb >> 31) mm = true; else pp = true; }
                                        if (nn || (pp && mm)) dn[r][c] = nan_bits;
                                        else if (pp || mm) dn[r][c] = pp ? 0x7F800000u : 0xFF800000u;
                                    }
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) d[r][c] = dn[r][c];
                    }
                    }
                }
                }
            };
            auto by_kind = [&](auto gl_c) {
                if (kind == 0) run_groups(gl_c, std::integral_constant<int, 0>{});
                else if (kind == 1) run_groups(gl_c, std::integral_constant<int, 1>{});
                else if (kind == 2) run_groups(gl_c, std::integral_constant<int, 2>{});
                else run_groups(gl_c, std::integral_constant<int, 3>{});
            };
            // End of a split group: T, the merged sum of the sub-groups in units of 2^(em - F_m) (hv: some product took
            // part); then as TR-FDPA with F_m in the place of F, rho, and Sec. 4.2's special values from the staged values
            // of the whole group of GLT terms at kg.
            auto finish_merged = [&](auto glt_c, uint32_t kg, const double (&T)[R][C], const bool (&hv)[R][C], const int (&em)[R][C],
                                     const uint32_t (&tg)[R][C], uint32_t tagged) {
                constexpr int GLT = decltype(glt_c)::value;
                slow_seen = true;
                uint32_t dn[R][C];
                double vrd[R][C];
                bool low = true;
                if (fl & FL_FTZ_IN) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) if ((d[r][c] & 0x7F800000u) == 0) d[r][c] = 0;             // FlushSubnormal on the accumulator
                }
                if (__builtin_expect((fl & FL_SUM_EXACT) != 0u, 0)) {
                    const double T4[4] = {T[0][0], T[0][1], T[1][0], T[1][1]};
                    const int e4[4] = {em[0][0], em[0][1], em[1][0], em[1][1]};
                    const uint32_t c4[4] = {d[0][0], d[0][1], d[1][0], d[1][1]};
                    double v[4];
                    low = rd_exact_all<false>(T4, e4, hot.Fm, c4, hot.F2, hot.Fc, hot.drop, fl, v);
                    vrd[0][0] = v[0]; vrd[0][1] = v[1]; vrd[1][0] = v[2]; vrd[1][1] = v[3];
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) vrd[r][c] = rd_general(T[r][c], hv[r][c], em[r][c], hot.Fm, d[r][c], hot.F2, hot.Fc, hot.drop, fl);
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) dn[r][c] = __float_as_uint((float)vrd[r][c]);
                if ((fl & (FL_RZ | FL_FTZ_OUT)) != 0u || (low && (fl & FL_ZERO_POSITIVE) != 0u)) convert_rare(vrd, dn);
                if (tagged) {
                    const uint2 sp = special_products<R, C, TI * VS, TJ * VS, TI * VSD, TJ * VSD, GLT>(av + kg, bv + kg, 2u);
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c)
                            if (tg[r][c]) {
                                const uint32_t i = r * C + c, cb = d[r][c];
                                bool nn = (sp.x >> i) & 1u, pp = (sp.y >> i) & 1u, mm = (sp.y >> (16 + i)) & 1u;
                                if ((cb & 0x7FFFFFFFu) > 0x7F800000u) nn = true;                           // the accumulator joins
                                else if ((cb & 0x7FFFFFFFu) == 0x7F800000u) { if (cb >> 31) mm = true; else pp = true; }
                                if (nn || (pp && mm)) dn[r][c] = nan_bits;
                                else if (pp || mm) dn[r][c] = pp ? 0x7F800000u : 0xFF800000u;
                            }
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) d[r][c] = dn[r][c];
            };
            // Split groups (Algorithm "GTR-FDPA", steps 3 to 5, with consecutive sub-groups): every sub-group of SL terms is
            // summed at its own maximum; the sums are rounded down to F_m bits at the largest maximum of the sub-groups
            // that hold a product and added; then as TR-FDPA with F_m in the place of F.
            auto run_split = [&](auto sl_c, auto ns_c) {
                constexpr int SL = decltype(sl_c)::value, NS = decltype(ns_c)::value, GLT = SL * NS;
                constexpr int US = (SL / 4 <= 2) ? 2 : 1;
                if constexpr (GLT <= KC && !ADAPT && FAM == 2) {
#pragma unroll 1
                for (int g = 0; g < KC / GLT; ++g) {
                    const uint32_t kg = g * GLT;
                    // the packed maximum of sub-group sg of the staged tile (SL terms), from the kept quarter maxima
                    auto sub_max = [&](int sg, int r, int c) -> uint32_t {
                        if constexpr (SL == 4) {
                            return (m2k[sg / 2][tid][r * C + c] >> (16 * (sg & 1))) & 0xFFFFu;
                        } else {
                            uint32_t x = m2k[sg * (SL / 8)][tid][r * C + c];
#pragma unroll
                            for (int i = 1; i < SL / 8; ++i) x = pk_max_u16(x, m2k[sg * (SL / 8) + i][tid][r * C + c]);
                            const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                            return lo > hi ? lo : hi;
                        }
                    };
                    int em[R][C];
                    uint32_t tg[R][C], have[R][C], tagged = 0;
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            tg[r][c] = 0;
                            have[r][c] = 0;
                            int best = 0, first = 0;
#pragma unroll
                            for (int q = 0; q < NS; ++q) {
                                const uint32_t e = sub_max(g * NS + q, r, c);
                                tg[r][c] |= e & 0xC000u;
                                tagged |= e;
                                const int eq = (int)e + ebase;
                                if (q == 0) first = eq;
                                if (!(fl & FL_SKIP_ZERO) || e >= 2 * ZBIAS) {
                                    best = (!have[r][c] || eq > best) ? eq : best;
                                    have[r][c] |= 1u << q;
                                }
                            }
                            em[r][c] = have[r][c] ? best : first;
                        }
                    tagged &= 0xC000u;
                    double Tm[R][C];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) Tm[r][c] = 0.0;
                    // (one sub-group at a time, its maximum read again: four sets of maxima and sums in flight cost registers)
#pragma unroll 1
                    for (int q = 0; q < NS; ++q) {
                        int32_t S32[R][C];
                        int eq[R][C];
                        float scale[R][C];
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                S32[r][c] = 0;
                                eq[r][c] = (int)sub_max(g * NS + q, r, c) + ebase;
                                int se = F + 127 - eq[r][c];                           // biased exponent of 2^(F - e_max)
                                se = se < 1 ? 1 : (se > 254 ? 254 : se);               // the clamps never change a truncated term
                                scale[r][c] = __uint_as_float((uint32_t)se << 23);
                            }
#pragma unroll US
                        for (int t = 0; t < SL; t += 4) {
                            float a[R][4], b[C][4];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const float4 v = *reinterpret_cast<const float4 *>(av + TI * r * VS + kg + q * SL + t);
                                a[r][0] = v.x; a[r][1] = v.y; a[r][2] = v.z; a[r][3] = v.w;
                            }
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                const float4 v = *reinterpret_cast<const float4 *>(bv + TJ * c * VS + kg + q * SL + t);
                                b[c][0] = v.x; b[c][1] = v.y; b[c][2] = v.z; b[c][3] = v.w;
                            }
#pragma unroll
                            for (int w = 0; w < 4; ++w)
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int c = 0; c < C; ++c) S32[r][c] += (int32_t)((a[r][w] * b[c][w]) * scale[r][c]);
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int c = 0; c < C; ++c)
                                if ((have[r][c] >> q) & 1u) Tm[r][c] += __builtin_floor(ldexp((double)S32[r][c], (eq[r][c] - F) - (em[r][c] - hot.Fm)));
                    }
                    bool hv[R][C];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) hv[r][c] = have[r][c] != 0;
                    finish_merged(std::integral_constant<int, GLT>{}, kg, Tm, hv, em, tg, tagged);
                }
                }
            };
            // Algorithm "GTR-FDPA": the even and the odd products of a group are aligned at their own maxima (which pass 1's
            // packed arithmetic keeps apart: even k in the low halves) and summed apart; then merged as above.
            auto run_even_odd = [&](auto gl_c) {
                constexpr int GL = decltype(gl_c)::value;
                constexpr int UE = (GL / 4 <= 2) ? 2 : 1;
                if constexpr (GL <= KC && !ADAPT && FAM == 3) {
#pragma unroll 1
                for (int g = 0; g < KC / GL; ++g) {
                    const uint32_t kg = g * GL;
                    int ee[R][C], eo[R][C];
                    uint32_t tg[R][C], tagged = 0;
                    bool he[R][C], ho[R][C];
                    float scale_e[R][C], scale_o[R][C];
                    int32_t Se[R][C], So[R][C];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            uint32_t x = m2k[g * (GL / 4)][tid][r * C + c];
#pragma unroll
                            for (int i = 1; i < GL / 4; ++i) x = pk_max_u16(x, m2k[g * (GL / 4) + i][tid][r * C + c]);
                            const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
                            tg[r][c] = x & SENTINEL_MASK;
                            tagged |= x;
                            ee[r][c] = (int)lo + ebase;
                            eo[r][c] = (int)hi + ebase;
                            he[r][c] = !(fl & FL_SKIP_ZERO) || lo >= 2 * ZBIAS;
                            ho[r][c] = !(fl & FL_SKIP_ZERO) || hi >= 2 * ZBIAS;
                            int se = F + 127 - ee[r][c], so = F + 127 - eo[r][c];
                            se = se < 1 ? 1 : (se > 254 ? 254 : se);                  // the clamps never change a truncated term
                            so = so < 1 ? 1 : (so > 254 ? 254 : so);
                            scale_e[r][c] = __uint_as_float((uint32_t)se << 23);
                            scale_o[r][c] = __uint_as_float((uint32_t)so << 23);
                            Se[r][c] = 0;
                            So[r][c] = 0;
                        }
                    tagged &= SENTINEL_MASK;
#pragma unroll UE
                    for (int t = 0; t < GL; t += 4) {
                        float a[R][4], b[C][4];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float4 v = *reinterpret_cast<const float4 *>(av + TI * r * VS + kg + t);
                            a[r][0] = v.x; a[r][1] = v.y; a[r][2] = v.z; a[r][3] = v.w;
                        }
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const float4 v = *reinterpret_cast<const float4 *>(bv + TJ * c * VS + kg + t);
                            b[c][0] = v.x; b[c][1] = v.y; b[c][2] = v.z; b[c][3] = v.w;
                        }
#pragma unroll
                        for (int w = 0; w < 4; ++w)
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int c = 0; c < C; ++c) {
                                    if (w & 1) So[r][c] += (int32_t)((a[r][w] * b[c][w]) * scale_o[r][c]);
                                    else Se[r][c] += (int32_t)((a[r][w] * b[c][w]) * scale_e[r][c]);
                                }
                    }
                    double T[R][C];
                    int em[R][C];
                    bool hv[R][C];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const bool h0 = he[r][c], h1 = ho[r][c];
                            em[r][c] = (h0 && h1) ? (ee[r][c] > eo[r][c] ? ee[r][c] : eo[r][c]) : (h0 ? ee[r][c] : eo[r][c]);
                            T[r][c] = 0.0;
                            if (h0) T[r][c] += __builtin_floor(ldexp((double)Se[r][c], (ee[r][c] - F) - (em[r][c] - hot.Fm)));
                            if (h1) T[r][c] += __builtin_floor(ldexp((double)So[r][c], (eo[r][c] - F) - (em[r][c] - hot.Fm)));
                            hv[r][c] = h0 || h1;
                        }
                    finish_merged(gl_c, kg, T, hv, em, tg, tagged);
                }
                }
            };
            if constexpr (FAM == 3) {
                if (L == 4) run_even_odd(std::integral_constant<int, 4>{});
                else if (L == 8) run_even_odd(std::integral_constant<int, 8>{});
                else if (L == 16) run_even_odd(std::integral_constant<int, 16>{});
                else run_even_odd(std::integral_constant<int, 32>{});
            } else if constexpr (FAM == 2) {
                const uint32_t parts = hot.parts, SLr = L / parts;              // sub-groups of a group, terms of a sub-group
                if (parts == 2) {
                    if (SLr == 4) run_split(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
                    else if (SLr == 8) run_split(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
                    else run_split(std::integral_constant<int, 16>{}, std::integral_constant<int, 2>{});
                } else {
                    if (SLr == 4) run_split(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
                    else run_split(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{});
                }
            } else {
            if (L == 4) by_kind(std::integral_constant<int, 4>{});
            else if (L == 8) by_kind(std::integral_constant<int, 8>{});
            else if (L == 16) by_kind(std::integral_constant<int, 16>{});
            else by_kind(std::integral_constant<int, 32>{});                 // (no code where KC is below 32)
            }

            // ---- this model's outputs against the reference ----
            // (a pair of twins: the first model's outputs were set aside; then the twin's, in the next place of the arrays)
            if constexpr (TWIN) {
                if (twin) {
                    account(mi, dfirst, write_nan(dfirst, nan_first));
                    ++mi;
                }
            }
            account(mi, d, slow_seen && write_nan(d, nan_bits));   // (the short route produces no NaN)
        }
        }
        set_f32_round_toward_zero(false);
        }
    }
    __syncthreads();
    // one global atomic per non-zero counter per workgroup; n_compared and bucket 0 are known up front: workgroup 0 adds
    // the whole count once, every workgroup takes its non-zero buckets back out of bucket 0
    unsigned long long *gst = reinterpret_cast<unsigned long long *>(sa->stats);
    for (uint32_t i = tid; i < count * 34u; i += 256) {
        const uint32_t mi = i / 34u, b = i - mi * 34u;
        unsigned long long *g = gst + (uint64_t)sa->slot[mi] * STATS_WORDS;
        if (b == 0) {
            uint32_t nonzero = 0, mism = 0;
            for (int bb = 1; bb < 34; ++bb)
                for (int cpy = 0; cpy < HC; ++cpy) nonzero += ml.hist[mi][bb == 33 ? 33 : 32 - bb][cpy];
            for (int cpy = 0; cpy < HC; ++cpy) mism += ml.hist[mi][32][cpy];        // differing patterns at distance 0
            mism += nonzero;
            const unsigned long long total = (unsigned long long)nitems * (TM * TN);
            if (blockIdx.x == 0) { atomicAdd(&g[0], total); atomicAdd(&g[5], total); }
            if (nonzero) atomicAdd(&g[5], 0ull - (unsigned long long)nonzero);
            if (mism) {
                atomicAdd(&g[1], (unsigned long long)mism);
                atomicMin(&g[3], ml.first[mi]);
            }
            if (ml.naneq[mi]) atomicAdd(&g[2], (unsigned long long)ml.naneq[mi]);
            if (ml.maxd[mi]) atomicMax(&g[4], (unsigned long long)ml.maxd[mi]);
        } else {
            uint32_t t = 0;
            for (int cpy = 0; cpy < HC; ++cpy) t += ml.hist[mi][b == 33 ? 33 : 32 - b][cpy];
            if (t) atomicAdd(&g[5 + b], (unsigned long long)t);
        }
    }
}

template <int TM, int KC, bool ADAPT, int FAM, bool TWIN = false>
static mmaemu_status launch_scan_cfg(const ScanArgs &sa, const void *A, const void *B, const uint32_t *C, uint64_t batch, hipStream_t s)
{
    constexpr int SLOTS = 256 / ((TM / 2) * (TM / 2));
    const uint64_t blocks = (batch + SLOTS - 1) / SLOTS;
    if (blocks > 0x7FFFFFFFull) { set_error("emulate_compare_many: too many blocks"); return MMAEMU_ERR_SHAPE; }
    if (blocks == 0) return MMAEMU_OK;
    // Persistent workgroups: one resident set makes equal passes, a grid of several rounds of it lets the dispatcher balance what the
    // passes' data make unequal.  Against more of them stand the ends: where outputs differ, a workgroup's counters go to the same few
    // cache lines as every other's, one workgroup after the other at about 0.06 us (FP8 16x16x16, two sets that differ on most outputs,
    // 2^15 tiles: 105, 149, 261, 504 us with 1024, 2048, 4096, 8192 workgroups; where nothing differs 8192 cost no more than 1024).
    // What stands beside that is the launch's arithmetic, k x passes x (sets + 1) per workgroup, the last for staging and decoding; the
    // lines below are where a round more is the faster one with outputs that differ: launches of 1 to 16 sets on 2^12 to 2^18 tiles
    // take 0.977 of the time that a fixed 2048 workgroups from 2^14 blocks on, one round below, take, and no more than 1.08 of it
    // (few sets on outputs that mostly agree: two T-FDPA sets of equal sums on 2^16 tiles 16x16x16 E4M3 x E5M2 130 -> 141 us; two of
    // different widths 180 -> 144).  Sixteen T-FDPA sets on 2^16 tiles FP8 702,
    // 673, 667, 700 us with one, two, four, eight rounds; BF16 1057, 992, 978, 992; sixteen TR-FDPA sets on 2^15 tiles FP16 514,
    // 481, 462, 461; four sets on 2^16 tiles FP8 249, 239, 321, 532.
    // (workgroups that a device holds at once, by device; threads that ask at the same time work out the same number)
    static std::atomic<uint32_t> resident[16];
    int dev = 0;
    MMAEMU_HIP(hipGetDevice(&dev));
    uint32_t res = dev < 16 ? resident[dev].load(std::memory_order_relaxed) : 0u;
    if (!res) {
        int per_cu = 0, cus = 0;
        MMAEMU_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, emulate_scan_kernel<TM, KC, ADAPT, FAM, TWIN>, 256, 0));
        MMAEMU_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        res = (uint32_t)(per_cu > 0 ? per_cu : 1) * (uint32_t)(cus > 0 ? cus : 1);
        if (dev < 16) resident[dev].store(res, std::memory_order_relaxed);
    }
    uint32_t grid = 0;
    for (uint32_t rounds = 8; rounds >= 1; rounds /= 2) {
        const uint64_t workgroups = (uint64_t)rounds * res, passes = (blocks + workgroups - 1) / workgroups;
        // (whole rounds; a single one takes just as many workgroups as make the same number of passes)
        grid = (uint32_t)(rounds > 1 ? workgroups : (blocks + passes - 1) / passes);
        const uint64_t work = (KC + (FAM == 0 ? 0u : 8u)) * (sa.count + 1ull);          // (binary64 group ends: like eight products more)
        if (work * passes >= (rounds == 8 ? 1000u : 600u) && workgroups < blocks) break;
    }
    hipLaunchKernelGGL((emulate_scan_kernel<TM, KC, ADAPT, FAM, TWIN>), dim3(grid), dim3(256), 0, s, sa, A, B, C, batch, (uint32_t)blocks);
    MMAEMU_HIP(hipGetLastError());
    set_last_kernel("multi x%u tiled %dx%d r2x2 kc=%d any L vm=%d%s", sa.count, TM, TM, KC, ADAPT ? 1 : 0, FAM == 1 ? " rd" : FAM == 4 ? " kept rd" : (FAM == 2 ? " rd split" : (FAM == 3 ? " rd even/odd" : (TWIN ? ", twins share sums" : ""))));
    return MMAEMU_OK;
}

// Whether the kernel takes a model, the model's arithmetic kind, and the class of models it can share a launch with:
// 0, T-FDPA with the accumulator inside the sum; 1, TR-FDPA (unsplit groups, any of the variation switches); 2 and 3,
// TR-FDPA sets that keep zero terms out of the exponent maxima (the staged exponents then differ), without and with
// FlushSubnormal on the inputs (which decides what a zero is); 4 to 6, the same three for groups split in halves or
// quarters; 7 to 9, for the even / odd split.  Whole 16x16x16, 16x16x32, 32x32x8 or 32x32x16 tiles of
// FP8 / FP16 / BF16 / FP6 / FP4 operands, group length 4, 8, 16 or 32, F up to 40.
bool scan_takes(const ModelArgs &p, uint32_t ta, uint32_t tb, uint32_t m, uint32_t n, uint32_t k, const void *A, const void *B, uint32_t &kind,
                uint32_t &cls)
{
    const bool bf16 = ta == MMAEMU_BF16 || tb == MMAEMU_BF16;
    if (p.flags & (FL_ACC16 | FL_NAN_PROPAGATE)) return false;
    if (p.c_mode == MMAEMU_C_IN_GROUP) {
        if (p.skip_zero_terms || p.zero_result_positive) return false;
        cls = 0;
    } else if (p.c_mode == MMAEMU_C_AFTER_RD && p.split == MMAEMU_SPLIT_NONE) {
        // (BF16 products of 2^128 and more that keep their values need the general kernel's integer range; the truncating
        // variant of the round-downs exists for the plain F2 rule)
        if ((p.wide_products && bf16) || (p.rd_toward_zero && p.f2_at_leading_bit)) return false;
        cls = p.skip_zero_terms ? (p.ftz_in ? 3u : 2u) : 1u;
    } else if (p.c_mode == MMAEMU_C_AFTER_RD && (p.split == MMAEMU_SPLIT_HALVES || p.split == MMAEMU_SPLIT_QUARTERS)) {
        // halves or quarters of at least four terms, each summed in 32 bits, from binary32 values
        const uint32_t parts = p.split == MMAEMU_SPLIT_HALVES ? 2u : 4u;
        if (bf16 || p.rd_toward_zero || p.F >= 30 || p.L < 4 * parts || ((uint64_t)(p.L / parts) << (p.F + 2)) > (1ull << 31)) return false;
        cls = 4u + (p.skip_zero_terms ? (p.ftz_in ? 2u : 1u) : 0u);
    } else if (p.c_mode == MMAEMU_C_AFTER_RD && p.split == MMAEMU_SPLIT_EVEN_ODD) {
        // the even and the odd products of a group (Algorithm "GTR-FDPA"), each summed in 32 bits, from binary32 values
        if (bf16 || p.rd_toward_zero || p.F >= 30 || ((uint64_t)(p.L / 2) << (p.F + 2)) > (1ull << 31)) return false;
        cls = 7u + (p.skip_zero_terms ? (p.ftz_in ? 2u : 1u) : 0u);
    } else {
        return false;
    }
    if (!((m == 16 && n == 16 && (k == 16 || k == 32)) || (m == 32 && n == 32 && (k == 8 || k == 16)))) return false;
    if (ta == MMAEMU_FP32 || tb == MMAEMU_FP32 || ta == MMAEMU_TF32 || tb == MMAEMU_TF32) return false;
    if ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 7) return false;
    if (p.F > 40) return false;
    if (!(p.L == 4 || p.L == 8 || p.L == 16 || p.L == 32) || p.L > k) return false;
    const uint64_t term = 1ull << (p.F + 2);                // |aligned term| < 2^(F+2)
    kind = p.F >= 30 ? 3u : ((uint64_t)p.L * term <= (1ull << 31) ? 0u : (4 * term <= (1ull << 31) ? 1u : 2u));
    return true;
}

// tiles of one group whose launch holds twins (models that differ only in the output conversion)
static mmaemu_status launch_scan_twins(const ScanArgs &sa, const void *A, const void *B, const uint32_t *Cm, uint32_t m, uint32_t n, uint32_t k,
                                       uint64_t batch, bool adapt, hipStream_t s)
{
    if (m == 16 && n == 16 && k == 16) return adapt ? launch_scan_cfg<16, 16, true, 0, true>(sa, A, B, Cm, batch, s) : launch_scan_cfg<16, 16, false, 0, true>(sa, A, B, Cm, batch, s);
    if (m == 32 && n == 32 && k == 8) return adapt ? launch_scan_cfg<32, 8, true, 0, true>(sa, A, B, Cm, batch, s) : launch_scan_cfg<32, 8, false, 0, true>(sa, A, B, Cm, batch, s);
    if (m == 16 && n == 16 && k == 32) return adapt ? launch_scan_cfg<16, 32, true, 0, true>(sa, A, B, Cm, batch, s) : launch_scan_cfg<16, 32, false, 0, true>(sa, A, B, Cm, batch, s);
    if (m == 32 && n == 32 && k == 16) return adapt ? launch_scan_cfg<32, 16, true, 0, true>(sa, A, B, Cm, batch, s) : launch_scan_cfg<32, 16, false, 0, true>(sa, A, B, Cm, batch, s);
    set_error("emulate_compare_many: no kernel for this shape");
    return MMAEMU_ERR_UNSUPPORTED;
}

template <int FAM>
static mmaemu_status launch_scan_shape(const ScanArgs &sa, const void *A, const void *B, const uint32_t *Cm, uint32_t m, uint32_t n, uint32_t k,
                                       uint64_t batch, bool adapt, hipStream_t s)
{
    if constexpr (FAM >= 2) {                    // (binary32 values only)
        if (m == 16 && n == 16 && k == 16) return launch_scan_cfg<16, 16, false, FAM>(sa, A, B, Cm, batch, s);
        if (m == 32 && n == 32 && k == 8) return launch_scan_cfg<32, 8, false, FAM>(sa, A, B, Cm, batch, s);
        if constexpr (FAM != 4) {
            if (m == 16 && n == 16 && k == 32) return launch_scan_cfg<16, 32, false, FAM>(sa, A, B, Cm, batch, s);
        }
        if (m == 32 && n == 32 && k == 16) return launch_scan_cfg<32, 16, false, FAM>(sa, A, B, Cm, batch, s);
    } else {
    if (m == 16 && n == 16 && k == 16) return adapt ? launch_scan_cfg<16, 16, true, FAM>(sa, A, B, Cm, batch, s) : launch_scan_cfg<16, 16, false, FAM>(sa, A, B, Cm, batch, s);
    if (m == 32 && n == 32 && k == 8) return adapt ? launch_scan_cfg<32, 8, true, FAM>(sa, A, B, Cm, batch, s) : launch_scan_cfg<32, 8, false, FAM>(sa, A, B, Cm, batch, s);
    if (m == 16 && n == 16 && k == 32) return adapt ? launch_scan_cfg<16, 32, true, FAM>(sa, A, B, Cm, batch, s) : launch_scan_cfg<16, 32, false, FAM>(sa, A, B, Cm, batch, s);
    if (m == 32 && n == 32 && k == 16) return adapt ? launch_scan_cfg<32, 16, true, FAM>(sa, A, B, Cm, batch, s) : launch_scan_cfg<32, 16, false, FAM>(sa, A, B, Cm, batch, s);
    }
    set_error("emulate_compare_many: no kernel for this shape");
    return MMAEMU_ERR_UNSUPPORTED;
}

mmaemu_status launch_scan(const MultiLaunch &ml, const void *A, const void *B, const void *C, uint32_t m, uint32_t n, uint32_t k,
                          uint64_t batch, uint32_t ta, uint32_t tb, hipStream_t s)
{
    ScanArgs sa = {};
    sa.ta = ta;
    sa.tb = tb;
    sa.zbias = (ml.cls >= 1 && (ml.cls - 1) % 3 != 0) ? ZBIAS : 0u;
    sa.ebase = 2 - fmt_info(ta).bias - fmt_info(tb).bias - 2 * (int)sa.zbias;
    sa.count = ml.count;
    sa.ref_is_first = ml.ref_is_first ? 1u : 0u;
    sa.dref = ml.dref;
    sa.dout = ml.dout;
    sa.out_stride = ml.out_stride;
    sa.index_base = ml.index_base;
    sa.stats = reinterpret_cast<uint64_t *>(ml.stats);
    // Order within the launch.  T-FDPA models on tiles of one group (L = k) that differ only in the output conversion
    // (rounding, E8M13, output flush, NaN pattern) are twins: the second is moved next to the first (never across the
    // line between sets that flush their inputs and sets that do not: twins agree on that), and the kernel computes
    // their common maximum and sum once.
    uint32_t order[MULTI_MAX], n_order = 0;
    bool placed[MULTI_MAX] = {}, twin_of_next[MULTI_MAX] = {};
    bool any_twin = false;
    const uint32_t conversion_only = FL_RZ | FL_FTZ_OUT;
    for (uint32_t i = 0; i < ml.count; ++i) {
        if (placed[i]) continue;
        placed[i] = true;
        order[n_order++] = i;
        const ModelArgs &p = ml.models[i];
        if (ml.cls != 0 || p.L != k) continue;
        for (uint32_t j = i + 1; j < ml.count; ++j) {
            const ModelArgs &q = ml.models[j];
            if (placed[j] || q.L != p.L || q.F != p.F || ml.kind[j] != ml.kind[i] || ((q.flags ^ p.flags) & ~conversion_only) != 0) continue;
            placed[j] = true;
            twin_of_next[n_order - 1] = true;
            order[n_order++] = j;
            any_twin = true;
            break;
        }
    }
    for (uint32_t q = 0; q < ml.count; ++q) {
        const uint32_t i = order[q];
        const ModelArgs &p = ml.models[i];
        sa.slot[q] = ml.slot[i];
        sa.hot[q] = ScanArgs::Hot{p.F, p.flags, p.out_mask, p.nan_bits, p.L, ml.kind[i], p.F2, p.Fc, p.sum_drop_distance, p.Fm,
                                  p.split == MMAEMU_SPLIT_QUARTERS ? 4u : 2u, twin_of_next[q] ? 1u : 0u};
    }
    const bool adapt = ta == MMAEMU_BF16 || tb == MMAEMU_BF16;
    const uint32_t *Cm = static_cast<const uint32_t *>(C);
    if (ml.cls == 0 && any_twin) return launch_scan_twins(sa, A, B, Cm, m, n, k, batch, adapt, s);
    if (ml.cls == 0) return launch_scan_shape<0>(sa, A, B, Cm, m, n, k, batch, adapt, s);
    // TR-FDPA with the products in registers from six sets on: forming them, and the registers they take, cost a launch of few sets more than
    // the models save.  gfx950's sets of several widths on 2^15 tiles of 16x16x16 FP16, N(0,1), products formed for every model and
    // kept, 1, 4, 6, 8, 12, 16 sets: 55, 166, 232, 281, 411, 525 us and 66, 172, 231, 270, 385, 487; all bit patterns 82, 283, 407, 505, 717,
    // 951 and 72, 194, 262, 315, 440, 567.  Other tiles, six and twelve sets, 2^13 of 32x32x8 169, 291 and 150, 268 (all bit patterns 280, 499 and
    // 190, 329), of 32x32x16 245, 433 and 227, 389 (440, 784 and 283, 479); FP8, FP6 and FP4 within 2 % of that.  Sets whose sums no
    // flag calls exact save less (cdna3's, 2^15 tiles of 16x16x16: 266, 470 and 269, 451; all bit patterns 458, 808 and 323, 550): six of
    // them on 3000 to 10000 such tiles take 1.02 to 1.10, sixteen 0.93 to 1.04; below 3000 tiles 1.00 to 1.04.
    if (ml.cls <= 3 && !adapt && k <= 16 && ml.count >= 6) return launch_scan_shape<4>(sa, A, B, Cm, m, n, k, batch, false, s);
    if (ml.cls <= 3) return launch_scan_shape<1>(sa, A, B, Cm, m, n, k, batch, adapt, s);
    if (ml.cls <= 6) return launch_scan_shape<2>(sa, A, B, Cm, m, n, k, batch, false, s);
    return launch_scan_shape<3>(sa, A, B, Cm, m, n, k, batch, false, s);
}

} // namespace mmaemu

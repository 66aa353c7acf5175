// The end of a TR-FDPA group in binary64, for the kernels that keep a group's sum there.
#pragma once
#include "emulate_tiled.hpp"

namespace mmaemu {

// Algorithm "TR-FDPA", steps 3 and 4, and the variations of it that the model switches name, in binary64 (every quantity
// is an integer of fewer than 53 bits times a power of two, hence exact): T counts units of 2^(em - F) (have_T: a product
// took part), cb is the accumulator; returns the exact value whose conversion is the group's result.
__device__ __forceinline__ double rd_value(double T, bool have_T, int em, int F, uint32_t cb, int F2, int Fc, int drop, uint32_t fl)
{
    const int Fmax = F2 > Fc ? F2 : Fc;
    const uint32_t Ec = (cb >> 23) & 0xFFu;
    const int ec = (int)(Ec ? Ec : 1u) - 127;
    const int E = have_T ? (ec > em ? ec : em) : ec;                      // the accumulator always takes part
    if (have_T && drop && E - em >= drop) have_T = false;                 // the product sum lies too far below: it drops out
    if (!have_T) T = 0.0;
    const double sc_exact = ldexp((double)__uint_as_float(cb), Fc - E);
    double sc = (fl & FL_RD_AS_RZ) ? __builtin_trunc(sc_exact) : __builtin_floor(sc_exact);     // RD_Fc(c at E), units of 2^(E - Fc)
    if ((fl & FL_SPECIAL_TRUNC) && ec < E - Fc - 1 && Ec != 0xFFu) sc = 0.0;                   // (an infinite or NaN accumulator stays)
    if (!(fl & FL_F2_LEADING)) {
        const double T_exact = ldexp(T, (em - F) - (E - F2));
        const double T2 = (fl & FL_RD_AS_RZ) ? __builtin_trunc(T_exact) : __builtin_floor(T_exact);   // RD_F2(T at E)
        return ldexp(ldexp(T2, Fmax - F2) + ldexp(sc, Fmax - Fc), E - Fmax);
    }
    // F2 counted from the leading bit of the exact two-term sum, held as s + err (Knuth's TwoSum; |err| is below half a
    // last place of s, far under the unit that is kept)
    const double a = ldexp(T, em - F), b = ldexp(sc, E - Fc);
    const double sm = a + b, bb = sm - a;
    const double err = (a - (sm - bb)) + (b - bb);
    const long long sbits = __double_as_longlong(sm);
    int lead = (int)((sbits >> 52) & 0x7FF) - 1023;
    const bool toward_zero = (err != 0.0) && ((err < 0.0) != (sm < 0.0));
    if ((sbits & 0xFFFFFFFFFFFFFll) == 0 && toward_zero) lead -= 1;        // just inside the binade below
    lead = lead < -126 ? -126 : lead;                                       // binary32's smallest normal exponent
    const int unit = lead - F2;
    double q = __builtin_floor(ldexp(sm, -unit));
    if (err < 0.0 && ldexp(q, unit) == sm) q -= 1.0;                        // s on the grid, the exact sum just below it
    return sm == 0.0 ? 0.0 : ldexp(q, unit);
}

} // namespace mmaemu

// sin and cos of the FP64 bin loops.  Plain arithmetic on doubles, so that a host compiler can take it too.
#pragma once

namespace smcgw {

// v with its sign turned by the top bit of t (the high word alone is touched).
__device__ __forceinline__ double with_sign(double v, unsigned t) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned hi = (unsigned)(b >> 32) ^ (t & 0x80000000u);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | (unsigned)b);
}

// sin and cos of x revolutions: the nearest quarter turn off, polynomials on an eighth
// of a turn to either side (interpolated at Chebyshev nodes: 1e-19 and 9e-18 from the
// functions).  The quarter turns' number sits in the low bits of r's sum with 1.5 2^52,
// and the turn is a swap and two sign bits.  2 pi enters in two parts; the rounding of the cosine's first coefficient,
// -2 pi^2, is made up for where it counts, at the range's end, by five units in the last place of the second: error
// 8.7e-17 at most, 2.8e-17 rms (1.03e-16 without; sincospi: 0.97e-16, and the rms within 0.04e-17), far below the
// phase's own rounding; the likelihood's
// against 64-bit sums is sincospi's (4.9e-14 at 16 s).  The plain
// bin loop is bound by its instructions: 142 a bin of two detectors with sincospi, 27 of
// them a detector's range checks and selections; 1001 particles of 2 x 32449 bins
// 150 -> 125 us.
__device__ __forceinline__ void sincos_rev(double x, double& s, double& c) {
    const double r = x - __builtin_rint(x);
    const double m = __builtin_fma(4.0, r, 0x1.8p52);
    const double z = __builtin_fma(-0.25, m - 0x1.8p52, r);
    const unsigned n = (unsigned)__builtin_bit_cast(unsigned long long, m);
    const double z2 = z * z;
    double p = __builtin_fma(z2, 0x1.e4a9d9166f052p+1, -0x1.e3027dea82bd7p+3);
    p = __builtin_fma(z2, p, 0x1.50783208843ebp+5);
    p = __builtin_fma(z2, p, -0x1.32d2cce500387p+6);
    p = __builtin_fma(z2, p, 0x1.466bc6775a476p+6);
    p = __builtin_fma(z2, p, -0x1.4abbce625be52p+5);
    p = __builtin_fma(z2, p, 0x1.1a62633145c07p-52);
    double q = __builtin_fma(z2, -0x1.b2f3eb054afcdp+0, 0x1.f9ce245cada0bp+2);
    q = __builtin_fma(z2, q, -0x1.a6d1eef479be1p+4);
    q = __builtin_fma(z2, q, 0x1.e1f5068688d5bp+5);
    q = __builtin_fma(z2, q, -0x1.55d3c7e3cb241p+6);
    q = __builtin_fma(z2, q, 0x1.03c1f081b5abbp+6);
    const double sz = __builtin_fma(z, 0x1.921fb54442d18p+2, z * p);
    const double cz = __builtin_fma(z, __builtin_fma(z, -0x1.3bd3cc9be45dep+4, z * z2 * q), 1.0);
    const double a = n & 1 ? cz : sz, b = n & 1 ? sz : cz;
    s = with_sign(a, n << 30);
    c = with_sign(b, (n + 1) << 30);
}

}  // namespace smcgw

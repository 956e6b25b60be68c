// sin and cos of the FP64 bin loops.  Plain arithmetic on doubles, so that a host compiler can take it too.
#pragma once

namespace smcgw {

// sin and cos of x revolutions: the nearest quarter turn off, polynomials on an eighth
// of a turn to either side (interpolated at Chebyshev nodes: 1e-19 and 9e-18 from the
// functions).  The quarter turns' number sits in the low bits of r's sum with 1.5 2^52,
// and the turn is a swap and two sign bits.  2 pi and 2 pi^2 enter in two parts each, which costs
// nothing: error 8.7e-17 at most, 2.7e-17 rms (1.03e-16 and 2.8e-17 with 2 pi^2 rounded; sincospi:
// 0.97e-16, and the rms within 0.04e-17), far below the phase's own rounding; the likelihood's
// against 64-bit sums is sincospi's (4.9e-14 at 16 s).  The plain
// bin loop is bound by its instructions: 142 a bin of two detectors with sincospi, 27 of
// them a detector's range checks and selections; 1001 particles of 2 x 32449 bins
// 150 -> 125 us.
__device__ __forceinline__ void sincos_rev(double x, double& s, double& c) {
    const double r = x - __builtin_rint(x);
    const double m = __builtin_fma(4.0, r, 0x1.8p52);
    const double z = __builtin_fma(-0.25, m - 0x1.8p52, r);
    const unsigned long long n = __builtin_bit_cast(unsigned long long, m);
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
    q = __builtin_fma(z2, q, 0x1.03c1f081b5ac0p+6);
    q = __builtin_fma(z2, q, -0x1.692b71366cc04p-50);
    const double sz = __builtin_fma(z, 0x1.921fb54442d18p+2, z * p);
    const double cz = __builtin_fma(z, __builtin_fma(z, -0x1.3bd3cc9be45dep+4, z * q), 1.0);
    const double a = n & 1 ? cz : sz, b = n & 1 ? sz : cz;
    s = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, a) ^ (n & 2) << 62);
    c = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, b) ^ ((n + 1) & 2) << 62);
}

}  // namespace smcgw

// fp64 helper of the Gaussian-mixture grouping (Algorithm 2): 2^z for z <= 0,
// cheaper than the general library routine.
//
// gmm_exp2_nonpos(z) = 2^z for z <= 0: the responsibilities of the E-step are
// 2^(l_k - max_j l_j) with base-2 log-densities l_k, so the argument is never
// positive.  Method: table-driven range reduction (Tang, Table-driven
// implementation of the exponential function in IEEE floating-point arithmetic,
// ACM TOMS 15, 1989).  n = rint(32 z) from the low bits of 32 z + 1.5 * 2^52, f
// = z - n / 32 in [-1/64, 1/64] (exact for |z| <= 1022); 2^(n mod 32 / 32) from a
// table of the nearest doubles and their relative errors, its exponent raised by
// n / 32 with an integer addition; 2^f - 1 = f (ln 2 + ... + (ln 2)^6 f^5 / 720)
// by Horner's rule with fused multiply-adds (truncation below 3.5e-18 on |f ln
// 2| <= 0.0109), the table's error added by the last of them; one more
// multiply-add joins them.  Only the last rounding (0.5 ulp) and 0.0109 times
// the roundings of the polynomial are left.  Eleven fp64 operations, where a
// degree-13 polynomial on [-1/2, 1/2] with ldexp took 18.  Arguments below -1022 are clamped there, so
// the result never leaves the normal range (2^-1022 instead of a subnormal or
// 0, a difference far below any value a normalised sum of responsibilities
// can resolve).  The function is exact at 0 and at negative integers.  Compiled
// for the host as well, where the same IEEE operations give the same bits, so
// it is checked against libm on the CPU.
#pragma once

#include <math.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define GPOEO_HD __host__ __device__
#else
#define GPOEO_HD
#endif

namespace gpoeo {

constexpr int kExp2Table = 32;

// 2^(j / 32): the double nearest the exact value, and the relative difference
// left to it.
struct Exp2Entry {
    double value, rest;
};
#if defined(__HIPCC__)
__device__
#endif
constexpr Exp2Entry kExp2[kExp2Table] = {
    {1.0, 0.0},
    {1.0218971486541166, 4.9997448722726326e-17},
    {1.0442737824274138, 8.189317638195515e-17},
    {1.0671404006768237, -7.402825309426177e-17},
    {1.0905077326652577, -2.7939114859515733e-17},
    {1.1143867425958924, 9.341710609905046e-17},
    {1.1387886347566916, 7.826573258636076e-17},
    {1.1637248587775775, 3.2904726646008416e-17},
    {1.189207115002721, 3.3484623336251524e-17},
    {1.215247359980469, -6.346552106729483e-17},
    {1.241857812073484, 3.750854201303127e-17},
    {1.2690509571917332, 2.1023049675215714e-18},
    {1.2968395546510096, 1.9572585293112036e-17},
    {1.3252366431597413, -2.1571477251208752e-17},
    {1.3542555469368927, 5.68648095791174e-17},
    {1.383909881963832, -4.8923067513522756e-17},
    {1.4142135623730951, -6.835808657661922e-17},
    {1.4451808069770467, -2.092304381843353e-17},
    {1.4768261459394993, -2.3591094770850053e-17},
    {1.5091644275934228, -6.735219232374683e-17},
    {1.5422108254079407, 5.1548301170786783e-17},
    {1.5759808451078865, -6.432131775424189e-18},
    {1.6104903319492543, 1.5341410053603723e-17},
    {1.645755478153965, -6.152602891550265e-17},
    {1.681792830507429, 4.875160526227062e-17},
    {1.718619298122478, -1.0772487078934056e-17},
    {1.7562521603732995, 1.685487290628973e-17},
    {1.7947090750031072, 1.01562190116415e-17},
    {1.8340080864093424, 1.790126907604513e-17},
    {1.8741676341103, -3.266924100901318e-17},
    {1.9152065613971474, -5.545065618639427e-17},
    {1.9571441241754002, 4.5784915277060095e-17},
};

// `table`: kExp2, or a copy of it (the kernel keeps one in LDS).
GPOEO_HD inline double gmm_exp2_nonpos(double z, const Exp2Entry* table) {
    // (ln 2)^n / n!, n = 1..6, each the double nearest the exact value
    constexpr double c1 = 0.6931471805599453, c2 = 0.24022650695910072, c3 = 0.05550410866482158,
                     c4 = 0.009618129107628477, c5 = 0.0013333558146428443, c6 = 0.0001540353039338161;
    constexpr double magic = 6755399441055744.0;   // 1.5 * 2^52
    z = fmax(z, -1022.0);
    const double s = fma(z, 32.0, magic);
    const double f = fma(s - magic, -1.0 / 32.0, z);
    uint64_t bits;
    __builtin_memcpy(&bits, &s, 8);
    const int32_t n = (int32_t)(uint32_t)bits;
    const Exp2Entry entry = table[n & (kExp2Table - 1)];
    double t = entry.value;
    __builtin_memcpy(&bits, &t, 8);
    bits += (uint64_t)((uint32_t)(n & ~(kExp2Table - 1)) << 15) << 32;   // exponent + n / 32
    __builtin_memcpy(&t, &bits, 8);
    double p = c6;
    p = fma(p, f, c5);
    p = fma(p, f, c4);
    p = fma(p, f, c3);
    p = fma(p, f, c2);
    p = fma(p, f, c1);
    return fma(t, fma(f, p, entry.rest), t);
}
GPOEO_HD inline double gmm_exp2_nonpos(double z) { return gmm_exp2_nonpos(z, kExp2); }

}  // namespace gpoeo

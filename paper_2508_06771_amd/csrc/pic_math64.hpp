// pic_math64.hpp -- binary64 elementary functions on the arguments the
// collision step meets, for the device (and, with plain C functions for the
// hardware's approximations, for a host build that checks them).
//
// The general library functions pay for arguments that never occur here: the
// angles lie in (0, 2 pi), the logarithm's argument is a 24-bit uniform, and
// the square roots and quotients are of positive normal numbers.  Without the
// large-angle reduction, the scaling steps and the division fix-ups, a
// Takizuka & Abe pair takes 226 binary64 instructions, and the ten-member lean
// pass spilled 84 bytes per thread instead of 228 (28 now, see M64_SC): 40.96M
// binary64 electrons in cells of 10,000 took 1,279 us instead of 1,535, in
// cells of 3,052 (12.5M) 268 instead of 326.  The half change of a pair is within 4.5e-16 of 64-bit
// extended arithmetic (rms over 3M pairs; 4.5e-16 with the C library too).
// Polynomial coefficients: Chebyshev fits in 60 digits of sin(y)/y and cos(y)
// on |y| <= pi/4 and of 2 atanh(s)/s on the logarithm's reduced range (errors
// 1e-17, 1e-18 and 4e-18 of the result).
#pragma once

#include <stdint.h>

#ifndef PIC_M64_HOST
#define PIC_M64_FN __device__ __forceinline__
#define PIC_M64_MEM __constant__
#define PIC_M64_OPAQUE(c) asm volatile("" : "+s"(c))
#define PIC_M64_RCP(x) __builtin_amdgcn_rcp(x)
#define PIC_M64_RSQ(x) __builtin_amdgcn_rsq(x)
#define PIC_M64_FREXP_MANT(x) __builtin_amdgcn_frexp_mant(x)
#define PIC_M64_FREXP_EXP(x) __builtin_amdgcn_frexp_exp(x)
#endif

// The polynomials' coefficients, sines' first: as constants of the code (MEM
// false; two instructions or a register pair each) or, where a kernel's
// registers are full, from memory through the scalar cache, by a pointer the
// compiler cannot see through (MEM; one scalar load for several).  MEM in the
// kernels of 1,024 threads that spill without it: the ten-member lean pass
// spills 28 bytes per thread instead of 84 (40.96M binary64 electrons in cells
// of 10,000: 1,247 us a step against 1,390; with weights, 5,000 members, 204
// against 334; segments of cells of 40,000 288 against 380).  Not where
// registers are left: with MEM cells of 3,052 took 341 us (322 without), of
// 1,500 818 (766), of 200 172 (161), and not in the one-workgroup kernel of the
// largest cells (20 of 20,000 with the correction 413 us, 399 without).
#define PIC_M64_SC_LIST \
    0x1.5e0af18733f9ep-33, -0x1.907d7aec5a8a3p-37, -0x1.ae600a926df9ap-26, \
    0x1.71de37961e4dcp-19, -0x1.a01a019e8357dp-13, 0x1.1111111110bb1p-7, \
    -0x1.5555555555555p-3, 0x1.1eeb68b109cf5p-29, -0x1.27e4fa17a41bfp-22, \
    0x1.a01a019f4e867p-16, -0x1.6c16c16c16966p-10, 0x1.5555555555555p-5
#define PIC_M64_LN_LIST \
    0x1.2b59b70eb76c6p-3, 0x1.39fe42e9d4a8ap-3, 0x1.7462b58e4403ap-3, \
    0x1.c71c62e26212ep-3, 0x1.2492492df3ba9p-2, 0x1.99999999952ccp-2, \
    0x1.5555555555558p-1
PIC_M64_MEM const double M64_SC[] = {PIC_M64_SC_LIST};
PIC_M64_MEM const double M64_LN[] = {PIC_M64_LN_LIST};

// The square root of a positive x whose fourth power is normal, correctly
// rounded but for about one argument in 10^9 (Goldschmidt from the hardware's
// approximation, two steps and a correction); r: its reciprocal within 2 ulp.
PIC_M64_FN double m64_sqrt(double x, double &r)
{
    const double y = PIC_M64_RSQ(x);
    double g = x * y, h = 0.5 * y;
    double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    r = h + h;
    return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

// 1 / x of a normal x whose reciprocal is normal, within 1 ulp.
PIC_M64_FN double m64_rcp(double x)
{
    double r = PIC_M64_RCP(x);
    r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    return r;
}

// a / b from r, 1 / b within 2 ulp: correctly rounded but for about one pair in 10^6.
PIC_M64_FN double m64_div(double a, double b, double r)
{
    const double q = a * r;
    return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}

// sin and cos of p in [0, 2 pi] within 1 ulp.  p minus the nearest multiple q of pi/2
// is exact in binary64 (both are multiples of a unit below 2^-52), the low word
// of q pi/2 is carried as a correction to first order.
PIC_M64_FN void m64_sincos_c(double p, double &s, double &co, const double *c)
{
    const double q = __builtin_rint(p * 0x1.45f306dc9c883p-1);
    const double a = __builtin_fma(-q, 0x1.921fb54442d18p+0, p);
    const double y = __builtin_fma(-q, 0x1.1a62633145c07p-54, a);
    const double yl = __builtin_fma(-q, 0x1.1a62633145c07p-54, a - y);
    const double z = y * y;
    double ps = c[0];
    ps = __builtin_fma(ps, z, c[2]);
    ps = __builtin_fma(ps, z, c[3]);
    ps = __builtin_fma(ps, z, c[4]);
    ps = __builtin_fma(ps, z, c[5]);
    ps = __builtin_fma(ps, z, c[6]);
    double pc = c[1];
    pc = __builtin_fma(pc, z, c[7]);
    pc = __builtin_fma(pc, z, c[8]);
    pc = __builtin_fma(pc, z, c[9]);
    pc = __builtin_fma(pc, z, c[10]);
    pc = __builtin_fma(pc, z, c[11]);
    // sin y + yl cos y, cos y - yl sin y
    const double hz = 0.5 * z;
    const double sy = y + __builtin_fma(y * z, ps, __builtin_fma(-hz, yl, yl));
    const double cy = 1.0 - (hz - __builtin_fma(z * z, pc, -y * yl));
    const int k = (int)q;
    const double u = (k & 1) ? cy : sy, v = (k & 1) ? sy : cy;
    s = (k & 2) ? -u : u;
    co = ((k + 1) & 2) ? -v : v;
}

template <bool MEM = false>
PIC_M64_FN void m64_sincos(double p, double &s, double &c)
{
    if constexpr (MEM) {
        const double *k = M64_SC;
        PIC_M64_OPAQUE(k);
        m64_sincos_c(p, s, c, k);
    } else {
        constexpr double k[] = {PIC_M64_SC_LIST};
        m64_sincos_c(p, s, c, k);
    }
}

// log of a normal x in (0, 1) within 1 ulp: x = 2^e (1 + f) with 1 + f in
// [sqrt(1/2), sqrt(2)), log(1 + f) = f - f^2/2 + t (f^2/2 + R), t = f / (2 + f),
// R = 2 atanh(t) / t - 2, ln 2 in two parts: the reduction that fdlibm's log
// publishes (Sun Microsystems, 1993), with a polynomial of its own and the
// rounding errors of f - f^2/2 and of e ln 2 + that carried along.
PIC_M64_FN double m64_log_c(double x, const double *c)
{
    double m = PIC_M64_FREXP_MANT(x);     // [1/2, 1)
    int e = PIC_M64_FREXP_EXP(x);
    const bool low = m < 0x1.6a09e667f3bcdp-1;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0;
    const double t = f * m64_rcp(2.0 + f);
    const double z = t * t, f2 = 0.5 * f, hf = f2 * f;
    double r = c[0];
    r = __builtin_fma(r, z, c[1]);
    r = __builtin_fma(r, z, c[2]);
    r = __builtin_fma(r, z, c[3]);
    r = __builtin_fma(r, z, c[4]);
    r = __builtin_fma(r, z, c[5]);
    r = __builtin_fma(r, z, c[6]);
    // f - f^2/2 and k ln 2 + that, with their rounding errors
    const double k = (double)e, kh = k * 0x1.62e42feep-1;
    const double d = f - hf, dl = (f - d) - hf - __builtin_fma(f2, f, -hf);
    const double hi = kh + d, hl = e ? (kh - hi) + d : 0.0;
    return hi + (__builtin_fma(t, __builtin_fma(r, z, hf), __builtin_fma(k, 0x1.a39ef35793c76p-33, dl)) + hl);
}

template <bool MEM = false>
PIC_M64_FN double m64_log(double x)
{
    if constexpr (MEM) {
        const double *k = M64_LN;
        PIC_M64_OPAQUE(k);
        return m64_log_c(x, k);
    } else {
        constexpr double k[] = {PIC_M64_LN_LIST};
        return m64_log_c(x, k);
    }
}

// Half of the Takizuka & Abe change of the relative velocity (ux, uy, uz) with
// s^2 = C / |u|^3, the deviate from the uniforms U1 and U2 and the azimuth
// 2 pi U3, in the order of operations of the definition (a later rounding
// difference grows by orders of magnitude within a hundred steps).  A velocity
// whose square leaves the safe range is scaled by a power of two.
template <bool MEM = false>
PIC_M64_FN void m64_ta_half(double ux, double uy, double uz, double C, double U1, double U2, double U3,
                            double &hx, double &hy, double &hz)
{
#pragma clang fp contract(off)
    constexpr double TWO_PI = 2.0 * 3.14159265358979323846;
    double uu = ux * ux + uy * uy + uz * uz;
    hx = hy = hz = 0.0;
    if (uu == 0.0) return;
    const bool axis = ux * ux + uy * uy == 0.0;   // along z: the azimuth counts from x
    int k = 0;
    if (!(uu > 0x1p-600 && uu < 0x1p600)) {
        const double big = __builtin_fmax(__builtin_fabs(ux), __builtin_fmax(__builtin_fabs(uy), __builtin_fabs(uz)));
        k = PIC_M64_FREXP_EXP(big);
        ux = __builtin_ldexp(ux, -k);
        uy = __builtin_ldexp(uy, -k);
        uz = __builtin_ldexp(uz, -k);
        uu = ux * ux + uy * uy + uz * uz;
    }
    double r;
    const double um = m64_sqrt(uu, r);
    double z = m64_sqrt(-2.0 * m64_log<MEM>(U1), r);
    double sn, cs;
    m64_sincos<MEM>(TWO_PI * U2, sn, cs);
    z *= cs;
    const double u3 = um * um * um;
    double s2 = m64_div(C, u3, m64_rcp(u3));
    if (k) s2 = __builtin_ldexp(s2, -3 * k);
    double d;
    if (s2 > 0x1p-900 && s2 < 0x1p900) {
        d = m64_sqrt(s2, r) * z;
    } else {
        // zero, without bound (the quotient's correction then has no value: the
        // bare product), or no number; a half change this small is beyond any use
        s2 = C * PIC_M64_RCP(u3);
        if (k) s2 = __builtin_ldexp(s2, -3 * k);
        d = __builtin_sqrt(s2) * z;
        d = d > 0x1p450 ? 0x1p450 : d < -0x1p450 ? -0x1p450 : d;
    }
    const double den = 1.0 + d * d;
    r = m64_rcp(den);
    const double sin_t = m64_div(2.0 * d, den, r);
    const double omc = m64_div(2.0 * d * d, den, r);
    m64_sincos<MEM>(TWO_PI * U3, sn, cs);
    const double up2 = ux * ux + uy * uy;
    if (!axis) {
        double px = ux, py = uy, p2 = up2;
        const bool low = up2 < 0x1p-900;
        if (low) {
            px = __builtin_ldexp(ux, 480);
            py = __builtin_ldexp(uy, 480);
            p2 = px * px + py * py;
        }
        double up = m64_sqrt(p2, r);
        const double ex = m64_div(px, up, r), ey = m64_div(py, up, r);
        if (low) up = __builtin_ldexp(up, -480);
        hx = ex * uz * sin_t * cs - ey * um * sin_t * sn - ux * omc;
        hy = ey * uz * sin_t * cs + ex * um * sin_t * sn - uy * omc;
        hz = -up * sin_t * cs - uz * omc;
    } else {
        hx = um * sin_t * cs;
        hy = um * sin_t * sn;
        hz = -uz * omc;
    }
    hx *= 0.5;
    hy *= 0.5;
    hz *= 0.5;
    if (k) {
        hx = __builtin_ldexp(hx, k);
        hy = __builtin_ldexp(hy, k);
        hz = __builtin_ldexp(hz, k);
    }
}

// The binary64 half change of a pair (pic_math64.hpp) on the host, against the
// plain formula in extended precision, where s^2 = C / |u|^3 is ordinary, zero,
// beyond binary64 or infinite.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#define PIC_M64_HOST
#define PIC_M64_FN static inline
#define PIC_M64_MEM static
#define PIC_M64_OPAQUE(c) (void)(c)
#define PIC_M64_RCP(x) (1.0 / (x))
#define PIC_M64_RSQ(x) (1.0 / sqrt(x))
static double mant(double x) { int e; return frexp(x, &e); }
static int expo(double x) { int e; frexp(x, &e); return e; }
#define PIC_M64_FREXP_MANT(x) mant(x)
#define PIC_M64_FREXP_EXP(x) expo(x)
#include "pic_math64.hpp"

typedef long double X;

static void plain(const double *u, double C, double U1, double U2, double U3, X *h)
{
    // the angles are 2 pi U rounded to binary64, as the definition has them
    const X p2 = 2.0 * 3.14159265358979323846 * U2, p3 = 2.0 * 3.14159265358979323846 * U3;
    const X x = u[0], y = u[1], z = u[2];
    const X um = sqrtl(x * x + y * y + z * z), up = sqrtl(x * x + y * y);
    h[0] = h[1] = h[2] = 0;
    if (um == 0) return;
    const X dev = sqrtl(-2 * logl(U1)) * cosl(p2);
    const X d = sqrtl((X)C / (um * um * um)) * dev;
    X st, omc;
    if (fabsl(d) < 1e2000L) {
        st = 2 * d / (1 + d * d);
        omc = 2 * d * d / (1 + d * d);
    } else {
        st = 0;
        omc = 2;
    }
    const X cp = cosl(p3), sp = sinl(p3);
    if (up > 0) {
        h[0] = 0.5L * (x / up * z * st * cp - y / up * um * st * sp - x * omc);
        h[1] = 0.5L * (y / up * z * st * cp + x / up * um * st * sp - y * omc);
        h[2] = 0.5L * (-up * st * cp - z * omc);
    } else {
        h[0] = 0.5L * um * st * cp;
        h[1] = 0.5L * um * st * sp;
        h[2] = -0.5L * z * omc;
    }
}

int main()
{
    srand(3);
    auto unit = []() { return (floor(16777216.0 * (rand() / (RAND_MAX + 1.0))) + 0.5) / 16777216.0; };
    const double Cs[] = {0.0, 1e-300, 1e-40, 1e-3, 1.0, 1e40, 1e150, 1e300, INFINITY};
    const double scales[] = {1e-100, 1e-80, 1e-30, 1.0, 1e30, 1e80, 1e100};
    double worst = 0.0;
    for (double C : Cs)
        for (double sc : scales)
            for (int i = 0; i < 2000; ++i) {
                const double u[3] = {sc * (i % 7 ? unit() - 0.5 : 0.0), sc * (i % 7 ? unit() - 0.5 : 0.0), sc * (unit() - 0.5)};
                const double U1 = unit(), U2 = unit(), U3 = unit();
                double hx, hy, hz;
                m64_ta_half(u[0], u[1], u[2], C, U1, U2, U3, hx, hy, hz);
                X r[3];
                plain(u, C, U1, U2, U3, r);
                const double um = sqrt(u[0] / sc * u[0] / sc + u[1] / sc * u[1] / sc + u[2] / sc * u[2] / sc) * sc;
                const double e = fmax(fabs((double)(hx - r[0])), fmax(fabs((double)(hy - r[1])), fabs((double)(hz - r[2])))) / um;
                if (!(e < 1e-14)) {
                    printf("C %g, |u| %g, error %g: %g %g %g, expected %Lg %Lg %Lg\n", C, um, e, hx, hy, hz, r[0], r[1], r[2]);
                    return 1;
                }
                worst = fmax(worst, e);
            }
    printf("math64 ok, worst %.2g of the relative speed\n", worst);
    return 0;
}

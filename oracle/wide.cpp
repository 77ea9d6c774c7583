// The CPU oracle in 80-bit arithmetic (test infrastructure): hydro_oracle.c
// compiled unchanged with `double` replaced by `long double`, so that the
// rounding error of an FP64 evaluation of L(U) can be measured.  Literal
// constant expressions (1.0/6.0, the Simpson weights) stay binary64: they are
// the scheme's constants.
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <cmath>

namespace {
#define double long double
#include "hydro_oracle.c"
#undef double
}  // namespace

extern "C" void wide_leaf_rhs(const double *P, double dx, const double *origin, double gamma, double omega,
                              double eta1, long double *dU)
{
    const long np = 7L * 2744;
    long double *Pw = (long double *)malloc(sizeof(long double) * np);
    for (long i = 0; i < np; ++i) Pw[i] = P[i];
    const long double org[3] = {origin[0], origin[1], origin[2]};
    oracle_phys ph;
    memset(&ph, 0, sizeof ph);
    ph.gamma = gamma;
    ph.omega = omega;
    ph.eta1 = eta1;
    ph.eta2 = 0.1;
    long double am;
    oracle_leaf_rhs(Pw, dx, org, &ph, dU, &am);
    free(Pw);
}

// Eigenvalue counts of symmetric tridiagonal matrices (host and device).
#pragma once

#include <math.h>

namespace ed {

// Squared off-diagonal entry for sturm_count, of a matrix scaled to a norm of about
// 1.  One below 1e-40 counts as 1e-40, which moves no eigenvalue by more than 1e-20:
// with every coupling nonzero two successive minors are never both zero, also
// where the matrix decouples and x is an eigenvalue of the leading block.
__host__ __device__ inline double sturm_b2(double b) { return fmax(b * b, 1e-40); }

// Number of eigenvalues below x of the tridiagonal matrix with diagonal al and
// squared off-diagonal b2 (sturm_b2), both scaled so that the matrix norm is about
// 1: sign changes of the leading principal minors p_i = (al_i - x) p_{i-1} -
// b2_{i-1} p_{i-2}, one dependent FMA per row (the ratio form q_i = p_i / p_{i-1}
// has a division).  A zero minor counts by its sign bit: its neighbours have
// opposite signs, so exactly one change is seen whatever that bit is.  A row shrinks
// the larger of the last two minors to no less than about 1e-41 of it, and every
// four rows the pair is scaled by a power of two that brings it back to about 1, so
// neither underflows away.
__host__ __device__ inline int sturm_count(const double *al, const double *b2, int m, double x) {
    double q = 1.0, p = al[0] - x;
    int c = signbit(p) ? 1 : 0;
    int i = 1;
    for (; i + 4 <= m; i += 4) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double n = fma(al[i + t] - x, p, -(b2[i + t - 1] * q));
            c += signbit(n) != signbit(p);
            q = p;
            p = n;
        }
        int e;
        (void)frexp(fmax(fabs(p), fabs(q)), &e);
        p = ldexp(p, -e);
        q = ldexp(q, -e);
    }
    for (; i < m; ++i) {
        const double n = fma(al[i] - x, p, -(b2[i - 1] * q));
        c += signbit(n) != signbit(p);
        q = p;
        p = n;
    }
    return c;
}

}  // namespace ed

// Lowest eigenpair of the m x m symmetric tridiagonal Lanczos matrix L of
// Alg. lanczos (diagonal alpha, off-diagonal beta), 1 <= m <= 64.  Shared by
// the host driver and the batched device solver.
//
// The paper obtains Ritz pairs by QR iteration (Sec. 3.4).  Only the lowest
// pair is needed, so this uses Sturm-sequence bisection for the eigenvalue
// (the number of negative pivots of L - x I equals the number of eigenvalues
// below x) and inverse iteration with a partially pivoted elimination of
// L - theta I for the vector; both are backward stable.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace pd {

__host__ __device__ inline int tridiag_count_below(int m, const double *a, const double *b, double x) {
    int cnt = 0;
    double q = a[0] - x;
    const double tiny = 1e-300;
    if (q == 0.0) q = -tiny;
    if (q < 0) ++cnt;
    for (int i = 1; i < m; ++i) {
        q = a[i] - x - b[i - 1] * b[i - 1] / q;
        if (q == 0.0) q = -tiny;
        if (q < 0) ++cnt;
    }
    return cnt;
}

// Solves (L - th I) z = r in place: Gaussian elimination with partial pivoting,
// which on a tridiagonal matrix only ever swaps neighbouring rows and leaves a
// diagonal u0 and two superdiagonals u1, u2 (m doubles of scratch each).  A
// pivot below `floor` is replaced by +-floor (L - th I is singular to working
// precision when th is an eigenvalue, which inverse iteration wants).
__host__ __device__ inline void tridiag_solve(int m, const double *a, const double *b, double th, double *u0,
                                              double *u1, double *u2, double *r, double floor) {
    // the row being eliminated from: p0 p1 (columns c, c + 1), p2
    double p0 = a[0] - th, p1 = m > 1 ? b[0] : 0.0, p2 = 0.0, rc = r[0];
    for (int c = 0; c < m; ++c) {
        if (c + 1 < m) {
            double n0 = b[c], n1 = a[c + 1] - th, n2 = c + 2 < m ? b[c + 1] : 0.0, rn = r[c + 1];
            if (fabs(n0) > fabs(p0)) {
                double t;
                t = p0, p0 = n0, n0 = t;
                t = p1, p1 = n1, n1 = t;
                t = p2, p2 = n2, n2 = t;
                t = rc, rc = rn, rn = t;
            }
            if (fabs(p0) < floor) p0 = p0 < 0 ? -floor : floor;
            const double f = n0 / p0;
            u0[c] = p0, u1[c] = p1, u2[c] = p2, r[c] = rc;
            p0 = n1 - f * p1;
            p1 = n2 - f * p2;
            p2 = 0.0;
            rc = rn - f * rc;
        } else {
            if (fabs(p0) < floor) p0 = p0 < 0 ? -floor : floor;
            u0[c] = p0, u1[c] = u2[c] = 0.0, r[c] = rc;
        }
    }
    double z1 = 0.0, z2 = 0.0;   // z[i + 1], z[i + 2]
    for (int i = m - 1; i >= 0; --i) {
        const double z = (r[i] - u1[i] * z1 - u2[i] * z2) / u0[i];
        r[i] = z;
        z2 = z1;
        z1 = z;
    }
}

// An interval that holds every eigenvalue, and the largest row sum.
__host__ __device__ inline void tridiag_bounds(int m, const double *alpha, const double *beta, double *lo_out,
                                               double *hi_out, double *norm_out) {
    double lo = alpha[0], hi = alpha[0], norm = 0.0;
    for (int i = 0; i < m; ++i) {
        double r = (i > 0 ? fabs(beta[i - 1]) : 0.0) + (i < m - 1 ? fabs(beta[i]) : 0.0);
        lo = fmin(lo, alpha[i] - r);
        hi = fmax(hi, alpha[i] + r);
        norm = fmax(norm, fabs(alpha[i]) + r);
    }
    *lo_out = lo - 1e-12 * (norm + 1.0);
    *hi_out = hi + 1e-12 * (norm + 1.0);
    *norm_out = norm;
}

// Unit y with y[0] >= 0 (the Ritz vector keeps q_1's sign) for the eigenvalue
// th: three steps of inverse iteration.  A: 3 m doubles of scratch, v: m.
__host__ __device__ inline int tridiag_vector(int m, const double *alpha, const double *beta, double th, double norm,
                                              double *y, double *A, double *v) {
    for (int i = 0; i < m; ++i) v[i] = (1.0 + 0.01 * i) / sqrt((double)m);
    for (int pass = 0; pass < 3; ++pass) {
        tridiag_solve(m, alpha, beta, th, A, A + m, A + 2 * m, v, 2.2e-16 * fmax(norm, 1e-300));
        double s = 0.0;
        for (int i = 0; i < m; ++i) s += v[i] * v[i];
        s = sqrt(s);
        if (!(s > 0.0) || !isfinite(s)) return -2;
        for (int i = 0; i < m; ++i) v[i] /= s;
    }
    const double sg = v[0] < 0 ? -1.0 : 1.0;
    for (int i = 0; i < m; ++i) y[i] = sg * v[i];
    return 0;
}

// theta and unit y.  A: 3 m doubles of scratch, v: m doubles of scratch.
// Returns 0 or < 0.
__host__ __device__ inline int tridiag_lowest_work(int m, const double *alpha, const double *beta, double *theta,
                                                   double *y, double *A, double *v) {
    if (m < 1 || m > 64) return -1;
    if (m == 1) {
        *theta = alpha[0];
        y[0] = 1.0;
        return 0;
    }
    double lo, hi, norm;
    tridiag_bounds(m, alpha, beta, &lo, &hi, &norm);
    for (int it = 0; it < 200; ++it) {
        double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (tridiag_count_below(m, alpha, beta, mid) >= 1) hi = mid; else lo = mid;
    }
    const double th = 0.5 * (lo + hi);
    *theta = th;
    return tridiag_vector(m, alpha, beta, th, norm, y, A, v);
}

#ifdef __HIP_DEVICE_COMPILE__
// The same, by the 64 lanes of a wave (all of them call it, and all get the
// return value): the interval is cut at 64 points at once instead of one, so
// some ten rounds of Sturm counts end at neighbouring numbers where
// bisection takes sixty.  Lane 0 then finds the vector.
__device__ inline int tridiag_lowest_wave(int m, const double *alpha, const double *beta, double *theta, double *y,
                                          double *A, double *v) {
    if (m < 1 || m > 64) return -1;
    const int lane = threadIdx.x & 63;
    if (m == 1) {
        if (lane == 0) {
            *theta = alpha[0];
            y[0] = 1.0;
        }
        return 0;
    }
    double lo, hi, norm;
    tridiag_bounds(m, alpha, beta, &lo, &hi, &norm);
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        // points that rounding puts on an end say nothing; the last one is the middle, which lies inside
        const double x = lane < 63 ? lo + (hi - lo) * ((lane + 1) * (1.0 / 64.0)) : mid;
        const bool inside = x > lo && x < hi;
        const bool below = inside && tridiag_count_below(m, alpha, beta, x) >= 1;
        double h = below ? x : hi, l = inside && !below ? x : lo;
        for (int o = 32; o > 0; o >>= 1) {
            h = fmin(h, __shfl_xor(h, o, 64));
            l = fmax(l, __shfl_xor(l, o, 64));
        }
        // counts that rounding leaves out of order around the eigenvalue: keep the upper part
        if (l >= h) l = lo;
        lo = l;
        hi = h;
    }
    const double th = 0.5 * (lo + hi);
    int st = 0;
    if (lane == 0) {
        *theta = th;
        st = tridiag_vector(m, alpha, beta, th, norm, y, A, v);
    }
    return __shfl(st, 0, 64);
}
#endif

}  // namespace pd

// Scalar pieces of the tridiagonal divide-and-conquer eigensolver (Cuppen's
// method with deflation and Gu-Eisenstat eigenvectors), written once for the
// device kernels of eig.hip.  Every function is plain sequential code over
// arrays, so the same definitions can be compiled for the host.
//
// One merge joins two blocks whose eigendecompositions are known:
//   T = diag(T1, T2) + rho u u^T,  rho = |beta| >= 0,
// where beta couples the last row of T1 and the first row of T2 and
// u = e_last + sign(beta) e_first (T1, T2 had |beta| taken off their facing
// diagonal entries).  With T1 = Q1 D1 Q1^T, T2 = Q2 D2 Q2^T this is
//   diag(Q1, Q2) (D + rho z z^T) diag(Q1, Q2)^T,  z = [Q1^T e_last; sign(beta) Q2^T e_first],
// and the eigenproblem of D + rho z z^T is solved here.
#pragma once

#ifndef ZOLO_HD
#define ZOLO_HD __host__ __device__
#endif

#include <cmath>

namespace zolo {
namespace dc {

constexpr double kEps = 1.1102230246251565e-16;   // unit roundoff 2^-53

// Deflation (the rules of Cuppen's method as refined by Dongarra and
// Sorensen), as a scan over the merged poles in ascending order.  The caller
// normalises z (||z|| = 1, rho -> rho ||z||^2) and sets
//   tol = 8 eps max(max |d|, rho max |z|),
// then calls step() for t = 0..k-1 with the t-th smallest pole and its z,
// and finish() once.  Outputs (positions t are sorted positions):
//   pole[u], zp[u], src[u] for u < K: remaining poles, strictly ascending,
//     with their z and sorted position;
//   src[u], dval[u] for K <= u < k: deflated eigenvalues and positions;
//   ri, rj, rc, rs [0..nrot): rotations of the columns at sorted positions
//     (q_i, q_j) <- (c q_i + s q_j, c q_j - s q_i), to apply in order.
struct DeflateScan {
    double rho, tol;
    int k, K, ndef, nrot, prev;
    double dprev, zprev, plast;   // plast: the last kept pole
    double *pole, *zp, *dval, *rc, *rs;
    int *src, *ri, *rj;

    ZOLO_HD void begin(int k_, double rho_, double tol_) {
        k = k_;
        rho = rho_;
        tol = tol_;
        K = ndef = nrot = 0;
        prev = -1;
        dprev = zprev = plast = 0.0;
    }
    // A rotation moves a pole by at most tol, so a kept pole can land on or
    // below its predecessor; it is then moved just above it (an eigenvalue
    // change below tol), which keeps the poles strictly ascending.
    ZOLO_HD void keep(int t, double d, double z) {
        if (K > 0 && !(d > plast)) d = nextafter(plast, INFINITY);
        pole[K] = plast = d;
        zp[K] = z;
        src[K] = t;
        ++K;
    }
    ZOLO_HD void drop(int t, double d) {
        src[k - 1 - ndef] = t;
        dval[k - 1 - ndef] = d;
        ++ndef;
    }
    ZOLO_HD void step(int t, double dc, double zc) {
        if (rho * fabs(zc) <= tol) {          // negligible coupling: eigenpair as is
            drop(t, dc);
            return;
        }
        // Far from the test below, |cs sn| = |z z_prev| / h^2, decided without the
        // root and the divisions (the scan is one thread's chain).
        if (prev >= 0 && fabs((dc - dprev) * zprev * zc) > 1.0000001 * tol * (zprev * zprev + zc * zc)) {
            keep(prev, dprev, zprev);
        } else if (prev >= 0) {
            // Two close poles: a rotation of their columns zeroes z_prev.
            const double h = hypot(zprev, zc);
            const double cs = zc / h, sn = -zprev / h;
            if (fabs((dc - dprev) * cs * sn) <= tol) {
                ri[nrot] = prev;
                rj[nrot] = t;
                rc[nrot] = cs;
                rs[nrot] = sn;
                ++nrot;
                drop(prev, dprev * cs * cs + dc * sn * sn);
                dc = dprev * sn * sn + dc * cs * cs;
                zc = h;
            } else {
                keep(prev, dprev, zprev);
            }
        }
        prev = t;
        dprev = dc;
        zprev = zc;
    }
    // Flushes the last candidate; returns K.
    ZOLO_HD int finish() {
        if (prev >= 0) keep(prev, dprev, zprev);
        return K;
    }
};

// Sums over the poles at a point x of the secular equation, x measured from
// an origin pole: f = 1/rho + sum_j z_j^2 / (delta_j - x), and the derivative
// split at pole t: dpsi over j <= t, dphi over j > t (both positive).
struct SecularSums {
    double f, dpsi, dphi;
};

// Bracketed rational iteration for one root.  The bracket [lo, hi] always
// holds the sign change of f and ends when its ends are neighbouring numbers,
// as plain bisection does.  Between evaluations the next point is the zero of
//   c + p / (delta_t - y) + q / (delta_{t+1} - y),
// fitted to the value and to the two parts of the derivative at x (the
// "middle way" of Li 1993; the last root has no pole to its right, q = 0).
// Once a step is a few units in the last place, points a few units further
// on the other side of the root close the bracket.  A point outside the
// bracket, or slow progress, falls back to the midpoint.
struct SecularIter {
    double lo, hi, x, probe;
    int steps;

    ZOLO_HD void begin(double lo_, double hi_) {
        lo = lo_;
        hi = hi_;
        x = probe = 0.0;
        steps = 0;
    }
    // False when the bracket is closed; otherwise x is the next point.
    ZOLO_HD bool next() {
        const double m = 0.5 * (lo + hi);
        if (!(m > lo && m < hi)) return false;
        if (!(x > lo && x < hi)) x = m;
        return true;
    }
    // The next point from the sums at x; dl = delta_t - x < 0 and
    // dr = delta_{t+1} - x > 0 (ignored for the last root).
    ZOLO_HD void propose(const SecularSums& s, double dl, double dr, bool last) {
        double eta;
        if (last) {
            eta = dl + s.dpsi * dl * dl / (s.f - dl * s.dpsi);
        } else {
            const double dd = dl * dr;
            const double a = (dl + dr) * s.f - dd * (s.dpsi + s.dphi), b = dd * s.f;
            const double c = s.f - dl * s.dpsi - dr * s.dphi;
            const double disc = sqrt(fmax(a * a - 4.0 * b * c, 0.0));
            eta = a <= 0.0 ? (a - disc) / (2.0 * c) : 2.0 * b / (a + disc);
        }
        const double ulp = 2.0 * kEps * fabs(x);
        ++steps;
        if (!(fabs(eta) > 2.0 * ulp)) {          // converged (or NaN): close the bracket
            if (probe == 0.0) probe = 2.0 * ulp;
            x = s.f > 0.0 ? x - probe : x + probe;
            probe *= 4.0;
        } else if (steps > 12 && (steps & 1)) {
            x = 0.5 * (lo + hi);
        } else {
            x += eta;
        }
    }
    ZOLO_HD void cut(double f) {
        if (f > 0.0) hi = x;
        else lo = x;
    }
};

// Root t (0 <= t < K) of the secular equation 1 + rho sum_j zp_j^2 / (pole_j - lambda) = 0
// with poles strictly increasing and rho > 0: lambda_t lies in (pole_t, pole_{t+1})
// (the last in (pole_{K-1}, pole_{K-1} + rho)).  lambda is returned as
// pole[*org] + *tau with the origin the nearer pole, so that the distances
// pole_j - lambda = (pole_j - pole_org) - tau keep their relative accuracy.
// sums(origin, x, t) gives the SecularSums at origin + x.
template <class Sums>
ZOLO_HD inline void secular_root(int K, const double* pole, double rho, int t, int* org, double* tau, Sums sums) {
    const bool last = t + 1 == K;
    const double left = pole[t];
    const double right = last ? pole[t] + rho : pole[t + 1];
    int o = t;
    SecularIter it;
    it.begin(0.0, right - left);
    if (!last) {
        // f at the midpoint, relative to the left pole, picks the origin.
        const double half = 0.5 * (right - left);
        const SecularSums s = sums(left, half, t);
        if (s.f < 0.0) {        // root in the right half: measure from pole_{t+1}
            o = t + 1;
            it.begin(-half, 0.0);
            it.x = -half;
        } else {
            it.begin(0.0, half);
            it.x = half;
        }
        it.propose(s, -half, half, false);
    }
    const double po = pole[o];
    for (int n = 0; n < 400 && it.next(); ++n) {
        const SecularSums s = sums(po, it.x, t);
        it.cut(s.f);
        it.propose(s, (left - po) - it.x, (right - po) - it.x, last);
    }
    *org = o;
    *tau = 0.5 * (it.lo + it.hi);
}

// pole_i - lambda_j for the root stored as (org_j, tau_j).
ZOLO_HD inline double pole_minus_root(const double* pole, int i, int org_j, double tau_j) {
    return (pole[i] - pole[org_j]) - tau_j;
}

// Gu-Eisenstat: the z that makes the computed roots the exact eigenvalues
// of diag(pole) + rho zh zh^T,
//   zh_i^2 = (lambda_{K-1} - pole_i) / rho * prod_{j<i} (lambda_j - pole_i)/(pole_j - pole_i)
//                                       * prod_{i<j<K} (lambda_{j-1} - pole_i)/(pole_j - pole_i),
// every factor positive by interlacing and the products' at most 1.  This is
// the product over j = first, first + step, ... of the factors of j != i.
ZOLO_HD inline double lowner_product(int K, const double* pole, const int* org, const double* tau, int i, int first,
                                     int step) {
    double p = 1.0;
    for (int j = first; j < K; j += step) {
        if (j == i) continue;
        const int r = j < i ? j : j - 1;
        p *= pole_minus_root(pole, i, org[r], tau[r]) / (pole[i] - pole[j]);
    }
    return p;
}

// zh_i from the whole product; the sign of zp_i.
ZOLO_HD inline double lowner_z(int K, const double* pole, double zp_i, double rho, const int* org, const double* tau,
                               int i, double product) {
    const double p = product * (-pole_minus_root(pole, i, org[K - 1], tau[K - 1]) / rho);
    const double v = sqrt(fmax(p, 0.0));
    return zp_i >= 0.0 ? v : -v;
}

}  // namespace dc
}  // namespace zolo

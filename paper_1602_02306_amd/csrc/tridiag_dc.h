// Eigenvalues of a symmetric tridiagonal matrix and the first (and last) row
// of its eigenvector matrix, by divide and conquer, one workgroup per matrix.
//
// Cuppen's tearing (Numer. Math. 36, 1981): every off-diagonal b_i (>= 0 here)
// is taken off the two diagonal entries it couples, so the matrix is a sum of
// 1 x 1 blocks and rank-one terms b_i v v^T, and blocks are merged in pairs.
// A merge is the eigenproblem of D + rho z z^T with z = (last row of the left
// block's vectors, first row of the right one's):
//   - entries with rho |z_i| below tolerance, and one of each pair of poles so
//     close that a rotation which clears its z changes D less than that, are
//     left as they are (deflation);
//   - the others are the roots of f(x) = 1 + rho sum z_i^2 / (d_i - x), one per
//     interval between poles: a thread per root, each as an offset from its
//     nearest pole, by the two-pole rational iteration of R.-C. Li ("Solving
//     secular equations stably and efficiently", 1993) with a bracket;
//   - the vectors' components come from the z for which the computed roots are
//     exact (Gu and Eisenstat, SIAM J. Matrix Anal. Appl. 15, 1994), so they
//     are orthogonal to rounding whatever the gaps.
// Only the rows that are asked for are carried through (first and last always,
// ROWS more for the block form), O(n^2) work in all, with n threads: implicit
// QR does as much in one sequential chain of rotations.
#pragma once
#include <float.h>

#include "device_common.h"

namespace ecnt {

template <int NMAX>
struct DcLds {
    double D[NMAX], F[NMAX], L[NMAX], Z[NMAX];   // blocks: values, first and last row; merge: active first
    double sd[NMAX], sz[NMAX], sf[NMAX], sl[NMAX];   // a merge's entries in ascending order
    double mu[NMAX], zh[NMAX];
    int perm[NMAX], src[NMAX], act[NMAX], org[NMAX], close[NMAX];
    int stray;   // a root's iteration ended at its limit
};

// 1/x for a finite normal x: the hardware estimate y0 and the series 1/(1 - e) =
// 1 + e + e^2 + ..., e = 1 - x y0, to second order
__device__ __forceinline__ double rcp_fast(double x)
{
    const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
    return fma(fma(e, e, e), y, y);
}

// Sum (product, count) over the P lanes that share an entry, P = 1, 2, 4, 8, by
// quad permutations and the half-row mirror: every lane gets the same value.
template <int P>
__device__ __forceinline__ double team_sum(double x)
{
    if constexpr (P >= 2) x += dpp_f64<0xB1>(x);
    if constexpr (P >= 4) x += dpp_f64<0x4E>(x);
    if constexpr (P >= 8) x += dpp_f64<0x141>(x);
    return x;
}
template <int P>
__device__ __forceinline__ double team_prod(double x)
{
    if constexpr (P >= 2) x *= dpp_f64<0xB1>(x);
    if constexpr (P >= 4) x *= dpp_f64<0x4E>(x);
    if constexpr (P >= 8) x *= dpp_f64<0x141>(x);
    return x;
}
template <int P>
__device__ __forceinline__ int team_count(int x)
{
    if constexpr (P >= 2) x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true);
    if constexpr (P >= 4) x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true);
    if constexpr (P >= 8) x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);
    return x;
}

// Root j of 1 + rho sum_i z_i^2 / (d_i - x) for ascending poles d_0..d_{K-1}: the
// pole it is measured from and the offset.  Lane p of the P that share the root
// takes the poles p, p + P, ...  False where the iteration ends at its limit (most
// roots take 2 to 8 steps; bracketed halving down to what deflation leaves takes
// about 50, 48 being the most over 12 million roots of glued, graded, clustered
// and random matrices).
template <int P>
__device__ __forceinline__ bool dc_secular(const double *d, const double *z, int K, int j, int p0, double rho,
                                           int &org, double &mu)
{
    org = j;
    if (K == 1) {
        mu = rho * z[0] * z[0];
        return true;
    }
    const bool last = j == K - 1;
    double lo, hi;
    if (!last) {
        const double mid = 0.5 * (d[j + 1] - d[j]);
        double f = 0.0;
#pragma unroll 4
        for (int i = p0; i < K; i += P) f += z[i] * z[i] * rcp_fast((d[i] - d[j]) - mid);
        f = team_sum<P>(f);
        const bool left = 1.0 + rho * f >= 0.0;
        org = left ? j : j + 1;
        lo = left ? 0.0 : -mid;
        hi = left ? mid : 0.0;
        mu = left ? mid : -mid;
    } else {
        double s = 0.0;
        for (int i = p0; i < K; i += P) s += z[i] * z[i];
        s = team_sum<P>(s);
        lo = 0.0;
        hi = rho * s * (1.0 + 4.0 * DBL_EPSILON);
        mu = 0.5 * hi;
    }
    const double d0 = d[org];
    for (int it = 0; it < 64; ++it) {
        // psi over the poles up to j, phi over the others (one loop: the
        // threads of a wavefront have different j)
        double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;
#pragma unroll 4
        for (int i = p0; i < K; i += P) {
            const double y = rcp_fast((d[i] - d0) - mu), t = z[i] * z[i] * y, u = t * y;
            const bool low = i <= j;
            psi += low ? t : 0.0;
            dpsi += low ? u : 0.0;
            phi += low ? 0.0 : t;
            dphi += low ? 0.0 : u;
        }
        psi = rho * team_sum<P>(psi);
        dpsi = rho * team_sum<P>(dpsi);
        phi = rho * team_sum<P>(phi);
        dphi = rho * team_sum<P>(dphi);
        const double f = 1.0 + psi + phi;
        if (fabs(f) <= 8.0 * DBL_EPSILON * (1.0 + fabs(psi) + fabs(phi))) return true;
        if (f < 0.0) lo = mu;
        else hi = mu;
        const double p = (d[j] - d0) - mu;
        double eta;
        if (!last) {
            const double q = (d[j + 1] - d0) - mu;
            const double c = f - p * dpsi - q * dphi, a = (p + q) * f - p * q * (dpsi + dphi), b = p * q * f;
            const double disc = sqrt(fmax(a * a - 4.0 * b * c, 0.0));
            eta = a <= 0.0 ? (a - disc) / (2.0 * c) : 2.0 * b / (a + disc);
        } else {
            eta = p + p * p * dpsi / (f - p * dpsi);
        }
        double x = mu + eta;
        if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);   // also where eta is not a number
        if (x == mu) return true;
        mu = x;
    }
    return false;
}

struct DcNoRows {
    __device__ void rotate(int, int, double, double) {}
    __device__ void copy(int) {}
    __device__ void clear() {}
    __device__ void add(int, double) {}
    __device__ void scale(double) {}
    __device__ void store(int) {}
};

// On return s.D[0..N-1] are the eigenvalues (in no order), s.F the entries of
// the first row of the eigenvector matrix, s.stray whether to report a failure.  a, b: LDS, with entries of
// magnitude at most 1, b >= 0.  NMAX >= N; the workgroup has P NMAX threads, P
// neighbouring ones per entry (their sums over the poles are short chains of
// dependent instructions, so more lanes mean less time as long as the chip has
// room); every thread must call.  `rows` (P = 1) carries further rows of some
// matrix W to W times the vectors.
template <int NMAX, int P, typename Rows>
__device__ __forceinline__ void tridiag_dc(int N, const double *a, const double *b, DcLds<NMAX> &s, Rows &rows)
{
    constexpr double tol = 4.0 * DBL_EPSILON;
    const int t = threadIdx.x / P, p0 = threadIdx.x % P;
    if (threadIdx.x == 0) s.stray = 0;
    __syncthreads();
    if (t < N && p0 == 0) {
        double d = a[t];
        if (t > 0) d -= b[t - 1];
        if (t + 1 < N) d -= b[t];
        s.D[t] = d;
        s.F[t] = 1.0;
        s.L[t] = 1.0;
    }
    for (int sz = 1; sz < N; sz *= 2) {
        const int lo = t / (2 * sz) * (2 * sz), mid = lo + sz, hi = min(lo + 2 * sz, N);
        const bool merge = t < N && mid < hi;
        const double rho = merge ? b[mid - 1] : 0.0;
        __syncthreads();
        // ascending order, z, and the rows of the merged block
        if (merge) {
            const double d = s.D[t];
            int r = 0;
#pragma unroll 4
            for (int j = lo + p0; j < hi; j += P) {
                const double dj = s.D[j];
                r += (dj < d || (dj == d && j < t)) ? 1 : 0;
            }
            r = lo + team_count<P>(r);
            const bool left = t < mid;
            const double z = left ? s.L[t] : s.F[t];
            if (p0 == 0) {
                s.sd[r] = d;
                s.sz[r] = z;
                s.sf[r] = left ? s.F[t] : 0.0;
                s.sl[r] = left ? 0.0 : s.L[t];
                s.perm[r] = t;
                s.act[r] = rho * fabs(z) > tol ? 1 : 0;
                if (t == lo) s.close[lo] = 0;
            }
        }
        __syncthreads();
        // close poles: is there a pair at all?
        if (merge && s.act[t]) {
            int n = t + 1;
            while (n < hi && !s.act[n]) ++n;
            if (n < hi) {
                const double z1 = s.sz[t], z2 = s.sz[n];
                if (fabs((s.sd[n] - s.sd[t]) * z1 * z2) <= tol * (z1 * z1 + z2 * z2)) s.close[lo] = 1;
            }
        }
        __syncthreads();
        if (merge && t == lo && p0 == 0 && s.close[lo]) {   // rare: one thread of the block, in order
            int prev = -1;
            for (int p = lo; p < hi; ++p) {
                if (!s.act[p]) continue;
                if (prev >= 0) {
                    const double z1 = s.sz[prev], z2 = s.sz[p], t2 = z1 * z1 + z2 * z2;
                    const double d1 = s.sd[prev], d2 = s.sd[p];
                    if (fabs((d2 - d1) * z1 * z2) <= tol * t2) {
                        const double tau = sqrt(t2), c = z2 / tau, g = -z1 / tau;
                        s.sz[p] = tau;
                        s.sz[prev] = 0.0;
                        s.act[prev] = 0;
                        const double f1 = s.sf[prev], f2 = s.sf[p], l1 = s.sl[prev], l2 = s.sl[p];
                        s.sf[prev] = c * f1 + g * f2;
                        s.sf[p] = c * f2 - g * f1;
                        s.sl[prev] = c * l1 + g * l2;
                        s.sl[p] = c * l2 - g * l1;
                        s.sd[prev] = d1 * c * c + d2 * g * g;
                        s.sd[p] = d1 * g * g + d2 * c * c;
                        rows.rotate(s.perm[prev], s.perm[p], c, g);
                    }
                }
                prev = p;
            }
        }
        __syncthreads();
        // the active entries first (ascending), then the others
        int K = 0;
        if (merge) {
            int before = 0;
#pragma unroll 4
            for (int j = lo + p0; j < hi; j += P) {
                const int v = s.act[j];
                K += v;
                before += j < t ? v : 0;
            }
            K = team_count<P>(K);
            before = team_count<P>(before);
            const int slot = s.act[t] ? lo + before : lo + K + (t - lo - before);
            if (p0 == 0) {
                s.D[slot] = s.sd[t];
                s.Z[slot] = s.sz[t];
                s.F[slot] = s.sf[t];
                s.L[slot] = s.sl[t];
                s.src[slot] = s.perm[t];
            }
        }
        __syncthreads();
        const bool root = merge && t - lo < K;
        double mu = 0.0;
        int org = 0;
        if (root) {
            const bool met = dc_secular<P>(s.D + lo, s.Z + lo, K, t - lo, p0, rho, org, mu);
            if (p0 == 0) {
                if (!met) s.stray = 1;
                s.mu[t] = mu;
                s.org[t] = lo + org;
            }
        }
        __syncthreads();
        if (root) {   // the z for which these roots are exact (up to a common factor)
            const double di = s.D[t];
            double p = p0 == 0 ? (s.D[s.org[lo + K - 1]] - di) + s.mu[lo + K - 1] : 1.0;
#pragma unroll 4
            for (int j = lo + p0; j < lo + K - 1; j += P) {
                const double lam = (s.D[s.org[j]] - di) + s.mu[j];
                p *= lam * rcp_fast((j < t ? s.D[j] : s.D[j + 1]) - di);
            }
            p = team_prod<P>(p);
            if (p0 == 0) s.zh[t] = copysign(sqrt(fabs(p)), s.Z[t]);
        }
        __syncthreads();
        double lam = 0.0, f = 0.0, l = 0.0;
        rows.clear();
        if (root) {
            const double d0 = s.D[lo + org];
            double nn = 0.0;
#pragma unroll 4
            for (int i = lo + p0; i < lo + K; i += P) {
                const double u = s.zh[i] * rcp_fast((s.D[i] - d0) - mu);
                nn = fma(u, u, nn);
                f = fma(u, s.F[i], f);
                l = fma(u, s.L[i], l);
                rows.add(s.src[i], u);
            }
            const double inv = 1.0 / sqrt(team_sum<P>(nn));
            f = team_sum<P>(f) * inv;
            l = team_sum<P>(l) * inv;
            rows.scale(inv);
            lam = d0 + mu;
        } else if (merge) {
            rows.copy(s.src[t]);
        }
        __syncthreads();
        if (root && p0 == 0) {
            s.D[t] = lam;
            s.F[t] = f;
            s.L[t] = l;
        }
        if (merge) rows.store(t);
    }
    __syncthreads();
}

}  // namespace ecnt

// Reverse-mode derivative of the erf-smoothed estimator.
//
// Forward, per column (probe j at shift tau), as computed by the forward
// kernels (q_l = sig_{l-1} * slot_{l-1}; Algorithm 1 with alpha_i taken first
// and one classical Gram-Schmidt pass, fused into one update):
//   y_i = C q_i,  w_i = y_i - beta_i q_{i-1},  g = Q_i^T w_i,  alpha_i = g[i],
//   p = Q_i^T q_i,  c = g - alpha_i (p - e_i),  r_i = w_i - Q_i c,
//   beta_{i+1} = |r_i|,  q_{i+1} = r_i / beta_{i+1},
//   s = nu * e_1^T S_w(J_k) e_1,  S_w(x) = erfc(x / w) / 2,
//   C = M (A - tau I) M,  A = L + diag(V),  M independent of V and tau.
// Reverse, for i = k..1 (bars are adjoints; all sums over l run to i):
//   rbar    = qbar_{i+1} / beta_{i+1} + betabar_{i+1} q_{i+1}
//             (betabar_{i+1} first decreased by qbar_{i+1}^T q_{i+1} / beta_{i+1})
//   cbar_l  = -q_l^T rbar,   alphabar = alphabar_J - (p - e_i)^T cbar
//   gbar    = cbar + alphabar e_i,   u = Q_i cbar
//   wbar    = rbar + Q_i gbar
//   qbar_l += gbar_l w_i - c_l rbar - alpha_i cbar_l q_i
//   qbar_i += alphabar w_i - alpha_i u          (through p = Q^T Q e_i and alpha_i = q_i^T w_i)
//   qbar_{i-1} -= beta_i wbar,  betabar_i -= wbar^T q_{i-1},  ybar = wbar,
//   qbar_i += C ybar,  Vbar += (M ybar) .* (M q_i),  taubar -= (M ybar)^T (M q_i)
// with alphabar_J, betabar of the tridiagonal step from Daleckii-Krein:
//   Jbar = sbar * nu * Z (S[1] o z z^T) Z^T,  z = first row of Z.
// M q_i is kept from the forward (one block vector per step); c and p - e_i
// of every step too (k x k per column each).
#include <float.h>

#include "device_common.h"
#include "ecount_internal.h"

namespace ecnt {

__device__ __forceinline__ double smooth_step(double th, double w) { return 0.5 * erfc(th / w); }
__device__ __forceinline__ double smooth_step_d(double th, double w)
{
    return -exp(-(th / w) * (th / w)) / (w * 1.7724538509055160273);   // sqrt(pi)
}

// ---- tridiagonal adjoint: full eigendecomposition of J_ku, then alphabar, betabar ----
// One wavefront per column (k <= 32): implicit QR with Wilkinson shifts as in
// the quadrature's wavefront form, every lane running the rotation chain and
// lane r carrying row r of Z through it (both halves of the wavefront repeat
// the rows).  Then, with F = S[1] o z z^T, u^(l) = F Z[l], lane a holding row a
// of F: alphabar_l = scale Z[l].u^(l), betabar_{l+1} = 2 scale Z[l-1].u^(l); the
// halves take even and odd l.  Bound: the sequential rotations (about 1.6 k^2).
// With a lane per column and Z in global memory 64 columns of k = 30 took 19 ms.
__global__ __launch_bounds__(64) void k_tridiag_bwd(int C, int k, int m, double smooth_w,
                                                    double g_out,
                                                    const double *__restrict__ alpha,
                                                    const double *__restrict__ beta,
                                                    const int32_t *__restrict__ kused,
                                                    const double *__restrict__ nu,
                                                    double *__restrict__ abar,
                                                    double *__restrict__ bbar,
                                                    int32_t *__restrict__ flags)
{
    __shared__ double A_[kBasisChunk + 1], B_[kBasisChunk + 1], Sv[kBasisChunk];
    __shared__ double Z_[kBasisChunk * 32];   // column b, row r at b * 32 + r
    const int c = blockIdx.x, lane = threadIdx.x, row = lane & 31, half = lane >> 5;
    const int N = kused[c];
    for (int i = lane; i <= k; i += 64) {
        if (i < k && (N < 1 || i >= N)) abar[(size_t)i * C + c] = 0.0;
        if (i == 0 || N < 1 || i >= N) bbar[(size_t)i * C + c] = 0.0;
    }
    if (N < 1) return;
    if (lane < N) {
        A_[lane] = alpha[(size_t)lane * C + c];
        B_[lane] = lane + 1 < N ? beta[(size_t)(lane + 1) * C + c] : 0.0;
    }
    for (int b = half; b < 32; b += 2) Z_[b * 32 + row] = b == row ? 1.0 : 0.0;
    __syncthreads();
    int hi = N - 1, iter = 0;
    bool failed = false;
    while (hi > 0) {
        if (fabs(B_[hi - 1]) <= DBL_EPSILON * (fabs(A_[hi - 1]) + fabs(A_[hi])) ||
            fabs(B_[hi - 1]) < DBL_MIN) {
            __syncthreads();
            B_[hi - 1] = 0.0;
            __syncthreads();
            --hi;
            continue;
        }
        int lo = 0;
        {
            const int i = hi - 1 - row;
            bool neg = false;
            if (i >= 1) {
                const double bl = fabs(B_[i - 1]);
                neg = bl <= DBL_EPSILON * (fabs(A_[i - 1]) + fabs(A_[i])) || bl < DBL_MIN;
            }
            const unsigned msk = (unsigned)__ballot(neg);
            if (msk) lo = hi - 1 - (__ffs((int)msk) - 1);
        }
        if (++iter > 60 * N) {
            failed = true;
            break;
        }
        const double bb = B_[hi - 1];
        const double d = 0.5 * (A_[hi - 1] - A_[hi]);
        const double den = d + copysign(hypot(d, bb), d);
        const double mu = A_[hi] - (den != 0.0 ? bb * bb / den : 0.0);
        double x = A_[lo] - mu, y = B_[lo];
        double ak = A_[lo], bk = B_[lo], zk = Z_[lo * 32 + row], nbk = bk;
        // values ahead of the rotation (written by no rotation before theirs)
        double a1 = A_[lo + 1], b1 = lo + 1 < hi ? B_[lo + 1] : 0.0, z1 = Z_[(lo + 1) * 32 + row];
        for (int kk = lo; kk < hi; ++kk) {
            const int nx = min(kk + 2, hi);
            const double a2 = A_[nx], b2 = nx < hi ? B_[nx] : 0.0, z2 = Z_[nx * 32 + row];
            const double q2 = x * x + y * y;
            const bool nz = q2 > 0.0;
            const double ir = rsqrt_pos(nz ? q2 : 1.0);
            const double r = nz ? q2 * ir : 0.0;
            const double cs = nz ? x * ir : 1.0;
            const double sn = nz ? y * ir : 0.0;
            if (kk > lo) B_[kk - 1] = r;
            A_[kk] = cs * cs * ak + 2.0 * cs * sn * bk + sn * sn * a1;
            const double na1 = sn * sn * ak - 2.0 * cs * sn * bk + cs * cs * a1;
            nbk = cs * sn * (a1 - ak) + (cs * cs - sn * sn) * bk;
            Z_[kk * 32 + row] = cs * zk + sn * z1;
            zk = -sn * zk + cs * z1;
            ak = na1;
            bk = cs * b1;
            x = nbk;
            y = sn * b1;
            a1 = a2;
            b1 = b2;
            z1 = z2;
        }
        A_[hi] = ak;
        B_[hi - 1] = nbk;
        Z_[hi * 32 + row] = zk;
        __syncthreads();
    }
    if (failed && lane == 0) atomicOr(&flags[1], 1);
    if (lane < N) Sv[lane] = smooth_step(A_[lane], smooth_w);
    __syncthreads();
    // seed: d estimate / d s_c = +-1/m (eta columns +, xi columns -)
    const double sbar = g_out * ((c >= m) ? 1.0 : -1.0) / (double)m;
    const double scale = sbar * nu[c];
    const bool live = row < N;
    const int ra = live ? row : 0;
    const double ta = A_[ra], sa = Sv[ra], za = live ? Z_[ra * 32] : 0.0;
    double F[32];
#pragma unroll
    for (int b = 0; b < 32; ++b) {
        const int rb = b < N ? b : 0;
        const double tb = A_[rb];
        double D;
        if (fabs(ta - tb) < 1e-8 * (1.0 + fabs(ta)))
            D = smooth_step_d(0.5 * (ta + tb), smooth_w);
        else
            D = (sa - Sv[rb]) / (ta - tb);
        F[b] = b < N ? D * za * Z_[rb * 32] : 0.0;
    }
    for (int l0 = 0; l0 < N; l0 += 2) {
        const int l = min(l0 + half, N - 1);   // the last odd one repeats a row and stores the same
        double u = 0.0;
#pragma unroll
        for (int b = 0; b < 32; ++b) u += F[b] * Z_[b * 32 + l];
        double diag = Z_[ra * 32 + l] * u, off = l > 0 ? Z_[ra * 32 + l - 1] * u : 0.0;
        diag = row_sum16(diag);
        off = row_sum16(off);
        diag += __shfl_xor(diag, 16, 64);
        off += __shfl_xor(off, 16, 64);
        if (row == 0) {
            abar[(size_t)l * C + c] = scale * diag;
            if (l > 0) bbar[(size_t)l * C + c] = 2.0 * scale * off;   // betabar_{l+1}
        }
    }
}

// ---- backward dots: raw[s] = slot_s . qbar_{i+1} (s = 0..i), raw[i+1+s] = slot_s . slot_i (s < i)
template <int NS>
__global__ __launch_bounds__(64) void k_bdots(int64_t n, int C, int nct, int64_t rpc,
                                              const double *__restrict__ basis,
                                              const double *__restrict__ qbar, size_t ss, int i,
                                              double *__restrict__ part)
{
    // NS = i + 1 slots (0..i)
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int ct = (int)(L % nct);
    const int64_t chunk = L / nct;
    const int c = ct * 64 + (int)threadIdx.x;
    if (c >= C) return;
    const int64_t r0 = chunk * rpc, r1 = min(n, r0 + rpc);
    double accD[NS], accE[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) accD[s] = accE[s] = 0.0;
    const double *QB = qbar + (size_t)i * ss;   // qbar_{i+1}
    for (int64_t r = r0; r < r1; ++r) {
        const size_t e = (size_t)r * C + c;
        double q[NS];
        const double qb = QB[e];
#pragma unroll
        for (int s = 0; s < NS; ++s) q[s] = basis[(size_t)s * ss + e];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            accD[s] += q[s] * qb;
            accE[s] += q[s] * q[NS - 1];
        }
    }
    double *P = part + (size_t)chunk * 64 * C + c;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        P[(size_t)s * C] = accD[s];
        if (s + 1 < NS) P[(size_t)(NS + s) * C] = accE[s];
    }
}

// sums[row][c] = sum over chunks of part[chunk][row][c]: a workgroup per row and
// 64 columns (a thread per sum, its 2048 chunks in sequence, took 0.5 ms)
__global__ __launch_bounds__(64 * kFinWaves) void k_rowsum(int C, int nchunk,
                                                           const double *__restrict__ part,
                                                           double *__restrict__ sums)
{
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const double t = block_chunk_sum(part, kPartRows, C, blockIdx.y, c, 0, nchunk, c < C);
    if (c < C && threadIdx.x < 64) sums[(size_t)blockIdx.y * C + c] = t;
}

// Per column: finish betabar_{i+1}, form the coefficients of rbar and gbar.
// coef layout (each [32][C]): cA = gbar*sig (wbar), cW = c*sig (w), cG = gbar, cR = c;
// scal[0][c] = a (qbar_{i+1} weight in rbar), scal[1][c] = b*sig_i (slot_i weight),
// scal[2][c] = -alpha_i sig_{i-1} (lambda: slot_{i-1} weight folded into w),
// scal[3][c] = alphabar sig_{i-1} (mu: slot_{i-1} weight of the alphabar term of wbar),
// scal[4][c] = -alpha_i.
__global__ __launch_bounds__(512) void k_bdots_fin(int C, int k, int i, int have_dots,
                            const double *__restrict__ sums, const double *__restrict__ sig,
                            const double *__restrict__ beta, const double *__restrict__ alpha,
                            const double *__restrict__ gall, const double *__restrict__ pall,
                            const double *__restrict__ abar, double *__restrict__ bbar,
                            const int32_t *__restrict__ kused, double *__restrict__ cA,
                            double *__restrict__ cW, double *__restrict__ cG,
                            double *__restrict__ cR, double *__restrict__ scal)
{
    // 64 columns; the slots of a column are spread over the 8 wavefronts
    __shared__ double red[8][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int craw = blockIdx.x * 64 + lane;
    const bool ok = craw < C;
    const int c = ok ? craw : C - 1;
    const int ku = kused[c];
    double a = 0.0, b = 0.0;
    const double sgi = sig[(size_t)i * C + c];
    auto raw = [&](int row) { return sums[(size_t)row * C + c]; };
    const bool on = have_dots && i < ku;
    if (on) {
        const double bi1 = beta[(size_t)i * C + c];                  // beta_{i+1}
        const double cc = sgi * raw(i);                              // qbar_{i+1}^T q_{i+1}
        a = 1.0 / bi1;
        b = bbar[(size_t)i * C + c] - cc / bi1;                      // betabar_{i+1}
    }
    auto cbar = [&](int s) {   // -q_s^T rbar
        if (a == 0.0 && b == 0.0) return 0.0;
        const double sg = sig[(size_t)s * C + c];
        return -(a * sg * raw(s) + b * sg * sgi * raw(i + 1 + s));
    };
    double t = 0.0;
    for (int s = wv; s < i; s += 8) t += pall[((size_t)(i - 1) * k + s) * C + c] * cbar(s);
    red[wv][lane] = t;
    __syncthreads();   // and every read of bbar above is done
    double ab = i <= ku ? abar[(size_t)(i - 1) * C + c] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) ab -= red[q][lane];
    if (!ok) return;
    for (int s = wv; s < i; s += 8) {
        const double sg = sig[(size_t)s * C + c];
        double gb = cbar(s);
        if (s == i - 1) gb += ab;
        const double cl = gall[((size_t)(i - 1) * k + s) * C + c];
        cA[(size_t)s * C + c] = gb * sg;
        cW[(size_t)s * C + c] = cl * sg;
        cG[(size_t)s * C + c] = gb;
        cR[(size_t)s * C + c] = cl;
    }
    if (wv != 0) return;
    if (on) bbar[(size_t)i * C + c] = b;
    const double al = alpha[(size_t)(i - 1) * C + c];
    const double sgq = sig[(size_t)(i - 1) * C + c];
    scal[c] = a;
    scal[(size_t)C + c] = b * sgi;
    scal[(size_t)2 * C + c] = -al * sgq;
    scal[(size_t)3 * C + c] = ab * sgq;
    scal[(size_t)4 * C + c] = -al;
}

// One sweep per row: rbar, wbar (= ybar) and w of step i, the partial
// wbar . slot_{i-2}, then qbar_s += cG_s (w - alpha_i q_i) - cR_s rbar (s < i),
// qbar_i += -alpha_i (u - alphabar q_i) (u = wbar - rbar - alphabar q_i) and
// qbar_{i-1} -= beta_i wbar.  rbar and w never leave registers.  A workgroup
// is four wavefronts on four row chunks of one column tile; they share the
// 4*NB coefficients of their columns through LDS.
template <int NB, bool HASQ, bool FIRST>
__global__ __launch_bounds__(256) void k_bupdate(int64_t n, int C, int nct, int64_t rpc,
                                                 int64_t nchunk, const double *__restrict__ basis,
                                                 double *__restrict__ qbar, size_t ss, int i,
                                                 const double *__restrict__ coef,
                                                 const double *__restrict__ scal,
                                                 const double *__restrict__ beta,
                                                 double *__restrict__ ybar,
                                                 double *__restrict__ part)
{
    // NB = i (slots 0..i-1), plus slot i.  coef: cA, cW, cG, cR, each [32][C]
    __shared__ double cf[4][NB][64];
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int ct = (int)(L % nct);
    const int64_t grp = L / nct;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = ct * 64 + lane;
    const bool colok = c < C;
    for (int idx = wv; idx < 4 * NB; idx += 4) {
        const int kind = idx / NB, s = idx - kind * NB;
        cf[kind][s][lane] = colok ? coef[((size_t)kind * 32 + s) * C + c] : 0.0;
    }
    __syncthreads();
    const int64_t chunk = grp * 4 + wv;
    if (!colok || chunk >= nchunk) return;
    const int64_t r0 = chunk * rpc, r1 = min(n, r0 + rpc);
    const double a = scal[c], bq = scal[(size_t)C + c];
    const double lam = scal[(size_t)2 * C + c], mu = scal[(size_t)3 * C + c];
    const double nal = scal[(size_t)4 * C + c];
    const double bi = i >= 2 ? beta[(size_t)(i - 1) * C + c] : 0.0;   // beta_i
    const double *QB = qbar + (size_t)i * ss;
    const double *SI = basis + (size_t)i * ss;
    const int sm = i >= 2 ? i - 2 : 0;
    double dotm = 0.0;
    for (int64_t r = r0; r < r1; ++r) {
        const size_t e = (size_t)r * C + c;
        double q[NB];
        const double si = SI[e];
        const double qb = HASQ ? QB[e] : 0.0;
#pragma unroll
        for (int s = 0; s < NB; ++s) q[s] = __builtin_nontemporal_load(basis + (size_t)s * ss + e);
        __builtin_amdgcn_sched_barrier(0);
        const double rb = a * qb + bq * si;
        double wb = rb, w = si;
#pragma unroll
        for (int s = 0; s < NB; ++s) {
            wb += cf[0][s][lane] * q[s];
            w += cf[1][s][lane] * q[s];
        }
        ybar[e] = wb;
        double qsm = 0.0;   // q[sm] by selects: a runtime index would move q to scratch
#pragma unroll
        for (int s = 0; s < NB; ++s) qsm = s == sm ? q[s] : qsm;
        dotm += wb * qsm;
        const double qi = q[NB - 1];                          // slot i-1 (q_i unnormalized)
        const double wq = w + lam * qi;                       // w - alpha_i q_i
        const double xq = nal * (wb - rb - 2.0 * mu * qi);    // -alpha_i (u - alphabar q_i)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NB; ++s) q[s] = FIRST ? 0.0 : qbar[(size_t)s * ss + e];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NB; ++s) {
            double v = q[s] + cf[2][s][lane] * wq - cf[3][s][lane] * rb;
            if (s == i - 2) v -= bi * wb;
            if (s == NB - 1) v += xq;
            qbar[(size_t)s * ss + e] = v;
        }
    }
    part[(size_t)chunk * 64 * C + c] = dotm;
}

// betabar_i -= sig_{i-2} * sum_chunks (wbar . slot_{i-2})
__global__ __launch_bounds__(64 * kFinWaves) void k_bnorm_fin(int C, int nchunk, int i,
                                                              const double *__restrict__ part,
                                                              const double *__restrict__ sig,
                                                              double *__restrict__ bbar)
{
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const double t = block_chunk_sum(part, kPartRows, C, 0, c, 0, nchunk, c < C);
    if (c < C && threadIdx.x < 64) bbar[(size_t)(i - 1) * C + c] -= sig[(size_t)(i - 2) * C + c] * t;
}

// Vbar and taubar contributions of step i: tb = M ybar_i, tq = M q_i.
// vpart[ct][r] (+)= sum over the tile's columns of tb*tq (in VALU, fixed
// order); part[chunk][0][c] = sum over the chunk's rows of tb*tq.  Four rows at
// a time; lane j < 4 keeps the sum of row r + j.
__global__ __launch_bounds__(64) void k_vgrad(int64_t n, int C, int nct, int64_t rpc,
                                              const double *__restrict__ tb,
                                              const double *__restrict__ tq, int first,
                                              double *__restrict__ vpart,
                                              double *__restrict__ part)
{
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int ct = (int)(L % nct);
    const int64_t chunk = L / nct;
    const int lane = threadIdx.x;
    const int craw = ct * 64 + lane;
    const bool ok = craw < C;
    const int c = ok ? craw : C - 1;
    const int64_t r0 = chunk * rpc, r1 = min(n, r0 + rpc);
    double tacc = 0.0;
    for (int64_t r = r0; r < r1; r += 4) {
        double *dst = vpart + (size_t)ct * n + r + lane;
        const bool mine = lane < 4 && r + lane < r1;
        const double old = (mine && !first) ? *dst : 0.0;
        double x[4], y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t e = (size_t)min(r + j, r1 - 1) * C + c;
            x[j] = tb[e];
            y[j] = tq[e];
        }
        double keep = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double p = (ok && r + j < r1) ? x[j] * y[j] : 0.0;
            tacc += p;
            const double t = wave_sum_dpp(p);
            keep = lane == j ? t : keep;
        }
        if (mine) *dst = old + keep;
    }
    if (ok) part[(size_t)chunk * kPartRows * C + c] = tacc;
}

__global__ __launch_bounds__(64 * kFinWaves) void k_vgrad_fin(int C, int nchunk,
                                                              const double *__restrict__ part,
                                                              double *__restrict__ taubar, int first)
{
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const double t = block_chunk_sum(part, kPartRows, C, 0, c, 0, nchunk, c < C);
    if (c < C && threadIdx.x < 64) taubar[c] = (first ? 0.0 : taubar[c]) - t;
}

// dV[r] = sum_ct vpart[ct][r]
__global__ void k_grad_v(int64_t n, int nct, const double *__restrict__ vpart, double *__restrict__ dV)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double t = 0.0;
    for (int ct = 0; ct < nct; ++ct) t += vpart[(size_t)ct * n + r];
    dV[r] = t;
}

// out[0] = sum of taubar over the xi columns, out[1] over the eta columns.
__global__ __launch_bounds__(256) void k_grad_tau(int m, const double *__restrict__ taubar,
                                                  double *__restrict__ out)
{
    __shared__ double sh[256];
    for (int s = 0; s < 2; ++s) {
        double acc = 0.0;
        for (int j = threadIdx.x; j < m; j += 256) acc += taubar[(size_t)s * m + j];
        sh[threadIdx.x] = acc;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[s] = sh[0];
        __syncthreads();
    }
}

// ------------------------------------------------------------------ launchers

static inline unsigned red_blocks(const Plan &p)
{
    const int nct = (p.C + 63) / 64;
    return (unsigned)((int64_t)p.nchunk * nct);
}

void launch_tridiag_bwd(const Plan &p, double g_out, hipStream_t st)
{
    k_tridiag_bwd<<<p.C, 64, 0, st>>>(p.C, p.k, p.m, p.smooth_w, g_out, p.alpha, p.beta, p.kused,
                                      p.nu, p.g_abar, p.g_bbar, p.flags);
}

#define ECNT_NS_CASES(F)                                                                        \
    F(1) F(2) F(3) F(4) F(5) F(6) F(7) F(8) F(9) F(10) F(11) F(12) F(13) F(14) F(15) F(16)   \
    F(17) F(18) F(19) F(20) F(21) F(22) F(23) F(24) F(25) F(26) F(27) F(28) F(29) F(30)     \
    F(31) F(32)

void launch_bdots(const Plan &p, int i, hipStream_t st)
{
    const int nct = (p.C + 63) / 64;
    const size_t ss = slot_elems(p);
    switch (i + 1) {
#define ECNT_CASE(N)                                                                             \
    case N:                                                                                      \
        k_bdots<N><<<red_blocks(p), 64, 0, st>>>(p.n, p.C, nct, p.rpc, (const double *)p.basis, \
                                                 p.g_qbar, ss, i, p.part);                       \
        break;
        ECNT_NS_CASES(ECNT_CASE)
#undef ECNT_CASE
    default:
        break;
    }
}

void launch_bdots_fin(const Plan &p, int i, bool have_dots, hipStream_t st)
{
    const size_t C = p.C;
    if (have_dots) {
        const int rows = 2 * i + 1;
        k_rowsum<<<dim3((p.C + 63) / 64, rows), 64 * kFinWaves, 0, st>>>(p.C, p.nchunk, p.part, p.g_sums);
    }
    k_bdots_fin<<<(p.C + 63) / 64, 512, 0, st>>>(p.C, p.k, i, have_dots ? 1 : 0,
                                                   p.g_sums, p.sig, p.beta, p.alpha, p.g_gall,
                                                   p.g_pall, p.g_abar,
                                                   p.g_bbar, p.kused, p.g_coef, p.g_coef + 32 * C,
                                                   p.g_coef + 64 * C, p.g_coef + 96 * C, p.g_scal);
}

void launch_bupdate(const Plan &p, int i, bool first, hipStream_t st)
{
    const int nct = (p.C + 63) / 64;
    const size_t ss = slot_elems(p);
    const size_t C = p.C;
    const bool hasq = i < p.k;
    (void)C;
    const dim3 grid((unsigned)(((int64_t)p.nchunk + 3) / 4 * nct));
    switch (i) {
#define ECNT_LAUNCH(N, HQ, FI)                                                                    \
    k_bupdate<N, HQ, FI><<<grid, 256, 0, st>>>(p.n, p.C, nct, p.rpc, (int64_t)p.nchunk,           \
                                               (const double *)p.basis, p.g_qbar, ss, i, p.g_coef, \
                                               p.g_scal, p.beta, p.g_ybar, p.part)
#define ECNT_CASE(N)                                                                              \
    case N:                                                                                       \
        if (hasq) {                                                                               \
            if (first) ECNT_LAUNCH(N, true, true);                                                \
            else ECNT_LAUNCH(N, true, false);                                                     \
        } else {                                                                                  \
            if (first) ECNT_LAUNCH(N, false, true);                                               \
            else ECNT_LAUNCH(N, false, false);                                                    \
        }                                                                                         \
        break;
        ECNT_NS_CASES(ECNT_CASE)
#undef ECNT_CASE
#undef ECNT_LAUNCH
    default:
        break;
    }
}

void launch_bnorm_fin(const Plan &p, int i, hipStream_t st)
{
    if (i < 2) return;   // beta_1 = 0 has no adjoint
    k_bnorm_fin<<<(p.C + 63) / 64, 64 * kFinWaves, 0, st>>>(p.C, p.nchunk, i, p.part, p.sig, p.g_bbar);
}

void launch_vgrad(const Plan &p, const double *tq, bool first, hipStream_t st)
{
    const int nct = (p.C + 63) / 64;
    k_vgrad<<<red_blocks(p), 64, 0, st>>>(p.n, p.C, nct, p.rpc, p.g_tbar, tq, first ? 1 : 0,
                                          p.g_vpart, p.part);
    k_vgrad_fin<<<(p.C + 63) / 64, 64 * kFinWaves, 0, st>>>(p.C, p.nchunk, p.part, p.g_taubar, first ? 1 : 0);
}

void launch_grad_out(const Plan &p, double *dV, hipStream_t st)
{
    const int nct = (p.C + 63) / 64;
    k_grad_v<<<(unsigned)((p.n + 255) / 256), 256, 0, st>>>(p.n, nct, p.g_vpart, dV);
    k_grad_tau<<<1, 256, 0, st>>>(p.m, p.g_taubar, p.result + 4 * kMaxShifts);
}

}  // namespace ecnt

// One-sweep Lanczos step: Algorithm 1 with full reorthogonalization at every
// step, reading the basis once per step instead of twice (k_lanczos.hip reads
// it for the dots and again for the update).
//
// The reorthogonalization of step i's vector is delayed past the operator: C
// is applied to the vector u_i that has only been taken through the
// three-term recurrence, and the sweep that finishes q_i also forms u_{i+1}
// and its dots with q_0..q_i.  With h = Q^T u_i (from the previous sweep) and
// z = C u_i, per column (indices from 0, beta_i couples q_{i-1} and q_i):
//   r      = u_i - Q h,          beta_i = |r|,  q_i = r / beta_i
//   C r    = z - C Q h = z - h_{i-1} u_i - Q t,    t = T h
//   alpha^ = r^T C r / beta_i^2   (u.z summed times a power of two, k_uz_scale)
//   u_{i+1} = C r / beta_i - alpha^ q_i - beta_i q_{i-1}
// where C Q h follows from the recurrence the basis satisfies (T the Lanczos
// matrix so far, its last column completed by u_i itself).  h is of the order
// of rounding (it is what the local recurrence loses in one step), so the
// second-order terms of C Q h that are dropped lie below rounding, and
// |r|^2 = |u_i|^2 - |h|^2 loses nothing.  alpha_i = alpha^ + h_i of the next
// step (the part of u_{i+1} left along q_i).  The basis stays orthogonal: every
// q_i has been orthogonalized against all of q_0..q_{i-1} before C q_i enters
// anything, and u_i was small against C q_{i-1} before that pass, not after it, so
// it also holds where the two-read form loses it (couplings below 1e-7 of the norm).
//
// Bound: HBM.  Step i reads i + 2 block vectors and writes 2, against 2i + 3
// read and 1 written for dots and update.  64^3 x 512 columns, k = 30: 116 ms
// (5.1 TB/s) and 11 ms for u.z, against 109 ms of updates (5.2 TB/s) and 81 ms
// of dots (6.6 TB/s); 32^3 x 64, k = 100: 18.5 ms against 33.1.
//
// Slots: 0..k-1 hold r_0.. (unnormalized, scales sig as in k_lanczos.hip);
// u_i lies in slot i until its sweep overwrites it with r_i; slot k holds z.
#include <float.h>

#include "device_common.h"
#include "ecount_internal.h"

namespace ecnt {

// Rows of the partial sums of a chunk: 0 u.u, 1 + l slot_l.u (l < i), i + 1 u.z;
// step 0: 0 v.v, 1 v.z, 2 z.z

// A power of two near 1 / sqrt(x) (1 where there is none).  u and z = C u are of
// the order of |C| and |C|^2 from step 1 on, so u.z would leave the range of a
// double at |C| = 2^340 already, where |u|^2 does at 2^511: its terms are taken
// times near 1 / |C|, in step 0 near 1 / |v|.
__device__ __forceinline__ double uz_scale(double x)
{
    return x > 0.0 && x <= DBL_MAX ? ldexp(1.0, -(ilogb(x) / 2)) : 1.0;
}

// scale[vc] for step 0, from the chunk sums of |v|^2 (row 0)
__global__ __launch_bounds__(64 * kFinWaves) void k_uz_scale(int C, int nseg, int rows,
                                                             const int64_t *__restrict__ seg_chunk,
                                                             const double *__restrict__ part,
                                                             double *__restrict__ scale)
{
    const int vc = blockIdx.x * 64 + (threadIdx.x & 63);
    const bool valid = vc < nseg * C;
    const int seg = valid ? vc / C : 0, c = valid ? vc - seg * C : 0;
    const double uu = block_chunk_sum(part, rows, C, 0, c, seg_chunk[seg], seg_chunk[seg + 1], valid);
    if (valid && threadIdx.x < 64) scale[vc] = uz_scale(uu);
}

// part[chunk][row][c] = scale * sum over the chunk's rows of U * Z; FIRST (step 0):
// and in the next row scale^2 * sum of Z * Z
template <bool FIRST>
__global__ __launch_bounds__(256) void k_dot_uz(int C, int nct, int64_t rpc, int nseg,
                                                const int64_t *__restrict__ seg_row,
                                                const int64_t *__restrict__ seg_chunk,
                                                const double *__restrict__ U,
                                                const double *__restrict__ Z,
                                                const double *__restrict__ scale, int rows, int row,
                                                double *__restrict__ part)
{
    __shared__ double red[4][64], red2[FIRST ? 4 : 1][64];
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int ct = (int)(L % nct);
    const int64_t chunk = L / nct;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = ct * 64 + lane;
    const int seg = find_seg(seg_chunk, nseg, chunk);
    const int64_t r0 = seg_row[seg] + (chunk - seg_chunk[seg]) * rpc;
    const int64_t r1 = min(seg_row[seg + 1], r0 + rpc);
    double a = 0.0, b = 0.0;
    if (c < C) {
        const double sc = scale[(size_t)seg * C + c];
        for (int64_t r = r0 + wv; r < r1; r += 4) {
            const size_t e = (size_t)r * C + c;
            const double z = Z[e];
            a += (U[e] * sc) * z;
            if (FIRST) b += (z * sc) * (z * sc);
        }
    }
    red[wv][lane] = a;
    if (FIRST) red2[FIRST ? wv : 0][lane] = b;
    __syncthreads();
    if (wv != 0 || c >= C) return;
    double *P = part + ((size_t)chunk * rows + row) * C + c;
    P[0] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if constexpr (FIRST) P[C] = (red2[0][lane] + red2[1][lane]) + (red2[2][lane] + red2[3][lane]);
}

// Chunk sums of rows 0..gridDim.y-1, each left in the segment's first chunk.
__global__ void k_sweep_sum(int C, int nseg, int rows, const int64_t *__restrict__ seg_chunk,
                            double *__restrict__ part)
{
    const int NC = nseg * C;
    const int vc = blockIdx.x * 64 + (threadIdx.x & 63);
    const bool valid = vc < NC;
    const int seg = valid ? vc / C : 0, c = valid ? vc - seg * C : 0;
    const int64_t ch0 = seg_chunk[seg], ch1 = seg_chunk[seg + 1];
    const double s = block_chunk_sum(part, rows, C, blockIdx.y, c, ch0, ch1, valid);
    if (valid && threadIdx.x < 64) part[((size_t)ch0 * rows + blockIdx.y) * C + c] = s;
}

// Scalars of step i per virtual column: beta_i, alpha_{i-1}, breakdown, and the
// coefficients of the sweep (cf: r -= cf_l slot_l; ec: u_{i+1} -= ec_l slot_l;
// cu, cr: the weights of u_i and r in u_{i+1}).  i = k: only beta_k and alpha_{k-1}.
__global__ __launch_bounds__(512) void k_sweep_fin(int C, int nseg, int rows, int i, int k,
                                                   double eps_vec,
                                                   const int64_t *__restrict__ seg_chunk,
                                                   const double *__restrict__ part,
                                                   double *__restrict__ scale,
                                                   double *__restrict__ nu, double *__restrict__ sig,
                                                   double *__restrict__ alpha,
                                                   double *__restrict__ beta,
                                                   double *__restrict__ cf, double *__restrict__ ec,
                                                   double *__restrict__ cu, double *__restrict__ cr,
                                                   double *__restrict__ runmax,
                                                   int32_t *__restrict__ active,
                                                   int32_t *__restrict__ kused, int ku_ld, int ku_off)
{
    extern __shared__ double sh[];   // h[i][64], then red[2][8][64]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int NC = nseg * C;
    const int vc = blockIdx.x * 64 + lane;
    const bool valid = vc < NC;
    const int v = valid ? vc : 0;
    const int seg = v / C, c = v - seg * C;
    const double *S = part + (size_t)seg_chunk[seg] * rows * C + c;
    auto at = [&](const double *a, int l) { return a[(size_t)l * NC + v]; };
    for (int l = w; l < i; l += 8) sh[l * 64 + lane] = S[(size_t)(1 + l) * C] * at(sig, l);
    __syncthreads();
    auto h = [&](int l) { return sh[l * 64 + lane]; };
    const double hl = i > 0 ? h(i - 1) : 0.0;
    const double a_last = i > 0 ? at(alpha, i - 1) + hl : 0.0;   // alpha_{i-1}
    auto tl = [&](int l) {
        double t = (l == i - 1 ? a_last : at(alpha, l)) * h(l);
        if (l + 1 < i) t += at(beta, l + 1) * h(l + 1);
        if (l >= 1) t += at(beta, l) * h(l - 1);
        return t;
    };
    const double sc = scale[v];   // of the sums u.z and h.t
    double hh = 0.0, ht = 0.0;
    for (int l = w; l < i; l += 8) {
        hh += h(l) * h(l);
        ht += (sc * h(l)) * tl(l);
    }
    double *red = sh + (size_t)i * 64;
    red[w * 64 + lane] = hh;
    red[(8 + w) * 64 + lane] = ht;
    __syncthreads();
    hh = ht = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        hh += red[q * 64 + lane];
        ht += red[(8 + q) * 64 + lane];
    }
    const double uu = S[0];
    const bool was = i == 0 ? uu > 0.0 : active[v] != 0;
    const double n2 = uu - hh <= 0.0 ? 0.0 : uu - hh, b = sqrt(n2);   // (not a number stays one)
    // the breakdown test of k_norm_fin
    double rm = 0.0;
    bool on = was;
    if (i > 0) {
        rm = fmax(runmax[v], was ? fabs(a_last) : 0.0);
        if (i > 1) rm = fmax(rm, at(beta, i - 1));
        on = was && !(b <= 1e3 * eps_vec * rm);
    }
    const double sg = on ? 1.0 / b : 0.0;
    const bool more = i < k;
    const double ah = (on && more) ? (S[(size_t)(i + 1) * C] - ht - 2.0 * (sc * hl) * uu) / (sc * n2) : 0.0;
    if (more && valid) {
        for (int l = w; l < i; l += 8) {
            const double sl = at(sig, l);
            cf[(size_t)l * NC + v] = on ? h(l) * sl : 0.0;
            ec[(size_t)l * NC + v] = on ? (sg * tl(l) + (l == i - 1 ? b : 0.0)) * sl : 0.0;
        }
    }
    // every read of the arrays written below is done
    __syncthreads();
    if (!valid || w != 0) return;
    if (i == 0) {
        nu[v] = uu;
        beta[v] = 0.0;
        kused[(size_t)seg * ku_ld + ku_off + c] = on ? k : 0;
        scale[v] = uz_scale(S[(size_t)2 * C]);   // |C v|^2 / |v|^2 to a factor of 4
    } else {
        alpha[(size_t)(i - 1) * NC + v] = was ? a_last : 0.0;
        beta[(size_t)i * NC + v] = was ? b : 0.0;
        if (was && !on) kused[(size_t)seg * ku_ld + ku_off + c] = i;
    }
    runmax[v] = rm;
    active[v] = on ? 1 : 0;
    sig[(size_t)i * NC + v] = sg;
    if (more) {
        alpha[(size_t)i * NC + v] = ah;
        cu[v] = sg * hl;
        cr[v] = ah * sg;
    }
}

// ---- the same for Arnoldi (two classical Gram-Schmidt passes per step) ----
// With w_i what the first pass left of C q_{i-1} and g' = Q^T w_i the second
// pass's dots, per column:
//   r = w_i - Q g',  h_{i, i-1} = |r|,  q_i = r / |r|
//   C r = z - C Q g' = z - Q (H g') - g'_{i-1} r,   z = C w_i
// so the sweep that finishes q_i also forms y = C q_i = C r / |r| and its dots
// g = Q^T y, and a second sweep takes the first pass, w_{i+1} = y - Q g, and the
// dots of the second, Q^T w_{i+1}: two reads of the basis per step, not four.
// g' is of the order of rounding, so |r|^2 = |w_i|^2 - |g'|^2.

// Before the first sweep of step i: column i - 1 of H, the breakdown test of
// k_arn_norm_fin, and the sweep's coefficients.  i = k: only the column.
__global__ __launch_bounds__(512) void k_arn_sweep_fin(int C, int nseg, int rows, int i, int k,
                                                       double eps_vec,
                                                       const int64_t *__restrict__ seg_chunk,
                                                       const double *__restrict__ part,
                                                       double *__restrict__ nu, double *__restrict__ sig,
                                                       double *__restrict__ H, double *__restrict__ cf,
                                                       double *__restrict__ ec, double *__restrict__ cu,
                                                       double *__restrict__ cr,
                                                       double *__restrict__ runmax,
                                                       int32_t *__restrict__ active,
                                                       int32_t *__restrict__ kused, int ku_ld, int ku_off)
{
    __shared__ double sh[kArnMaxK][64], red[2][8][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int NC = nseg * C;
    const int vc = blockIdx.x * 64 + lane;
    const bool valid = vc < NC;
    const int v = valid ? vc : 0;
    const int seg = v / C, c = v - seg * C;
    const double *S = part + (size_t)seg_chunk[seg] * rows * C + c;
    auto h = [&](int col, int row) -> double & { return H[((size_t)col * (k + 1) + row) * NC + v]; };
    const double uu = S[0];
    const bool was = i == 0 ? uu > 0.0 : active[v] != 0;
    double hh = 0.0, hm = 0.0;
    for (int l = w; l < i; l += 8) {
        const double g = was ? S[(size_t)(1 + l) * C] * sig[(size_t)l * NC + v] : 0.0;
        sh[l][lane] = g;
        const double x = h(i - 1, l) + g;
        if (valid) h(i - 1, l) = x;
        hh += g * g;
        hm = fmax(hm, fabs(x));
    }
    red[0][w][lane] = hh;
    red[1][w][lane] = hm;
    __syncthreads();
    hh = hm = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        hh += red[0][q][lane];
        hm = fmax(hm, red[1][q][lane]);
    }
    const double n2 = uu - hh <= 0.0 ? 0.0 : uu - hh, b = sqrt(n2);   // (not a number stays one)
    double rm = i > 0 ? fmax(runmax[v], hm) : 0.0;
    const bool on = was && (i == 0 || !(b <= 1e3 * eps_vec * rm));
    const double sg = on ? 1.0 / b : 0.0;
    if (on && i > 0) rm = fmax(rm, b);
    const bool more = i < k;
    if (more && valid) {
        for (int l = w; l < i; l += 8) {
            double t = 0.0;   // (H g')_l; column i - 1 was written by this thread
            for (int m = l > 0 ? l - 1 : 0; m < i; ++m) t += h(m, l) * sh[m][lane];
            const double sl = sig[(size_t)l * NC + v];
            cf[(size_t)l * NC + v] = on ? sh[l][lane] * sl : 0.0;
            ec[(size_t)l * NC + v] = on ? sg * t * sl : 0.0;
        }
    }
    __syncthreads();   // every read of what is written below is done
    if (!valid || w != 0) return;
    if (i == 0) {
        nu[v] = uu;
        kused[(size_t)seg * ku_ld + ku_off + c] = on ? k : 0;
    } else {
        h(i - 1, i) = was ? b : 0.0;
        if (was && !on) kused[(size_t)seg * ku_ld + ku_off + c] = i;
    }
    runmax[v] = rm;
    active[v] = on ? 1 : 0;
    sig[(size_t)i * NC + v] = sg;
    if (more) {
        cu[v] = 0.0;
        cr[v] = i > 0 ? sg * sh[i - 1][lane] : 0.0;
    }
}

// Before the second sweep of step i: g_l = q_l^T y, l = 0..i (row 1 + l).
__global__ __launch_bounds__(64 * kFinWaves) void k_arn_dots_fin(int C, int nseg, int rows, int i, int k,
                                                                 const int64_t *__restrict__ seg_chunk,
                                                                 const double *__restrict__ part,
                                                                 const double *__restrict__ sig,
                                                                 const int32_t *__restrict__ active,
                                                                 double *__restrict__ cf,
                                                                 double *__restrict__ H)
{
    const int NC = nseg * C;
    const int l = blockIdx.y;
    const int vc = blockIdx.x * 64 + (threadIdx.x & 63);
    const bool valid = vc < NC;
    const int seg = valid ? vc / C : 0, c = valid ? vc - seg * C : 0;
    const double s = block_chunk_sum(part, rows, C, 1 + l, c, seg_chunk[seg], seg_chunk[seg + 1], valid);
    if (!valid || threadIdx.x >= 64) return;
    const double sg = sig[(size_t)l * NC + vc];
    const double g = active[vc] ? s * sg : 0.0;
    cf[(size_t)l * NC + vc] = g * sg;
    H[((size_t)i * (k + 1) + l) * NC + vc] = g;
}

// The sweep of step i.  A workgroup of W wavefronts takes one row chunk of one
// 64-column tile; wavefront w owns slots w*NB.. (at most NB of the i), its
// coefficients and running dots in registers.  Per R rows each wavefront adds
// its slots' part of r and u_{i+1}; the parts meet in LDS (one barrier, two
// buffers), every wavefront forms the same r and u_{i+1} and takes the dots
// with its own slots, which are still in registers.  PLAIN: r alone, and the
// dots with r itself (a Gram-Schmidt pass and the next one's dots in one read).
template <int NB, int R, bool PLAIN, int WMAX>
__global__ __launch_bounds__(64 * WMAX) void k_sweep(int C, int nct, int64_t rpc, int nseg,
                                               const int64_t *__restrict__ seg_row,
                                               const int64_t *__restrict__ seg_chunk,
                                               double *__restrict__ basis, size_t ss, int i,
                                               const double *__restrict__ Z,
                                               const double *__restrict__ sig,
                                               const double *__restrict__ cf,
                                               const double *__restrict__ ec,
                                               const double *__restrict__ cu,
                                               const double *__restrict__ cr, int store_u, int rows,
                                               double *__restrict__ part)
{
    extern __shared__ double2 xch[];   // [2][W][R][64], W <= WMAX
    constexpr int NA = NB > 0 ? NB : 1;
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int ct = (int)(L % nct);
    const int64_t chunk = L / nct;
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6), W = uniform(blockDim.x >> 6);
    const int craw = ct * 64 + lane;
    const bool colok = craw < C;
    const int c = colok ? craw : C - 1;   // lanes past the last column repeat it and store nothing
    const int seg = find_seg(seg_chunk, nseg, chunk);
    const int64_t r0 = seg_row[seg] + (chunk - seg_chunk[seg]) * rpc;
    const int64_t r1 = min(seg_row[seg + 1], r0 + rpc);
    const size_t NC = (size_t)nseg * C, vc = (size_t)seg * C + c;
    const int l0 = w * NB, nb = min(NB, i - l0);   // nb < NB only in the last wavefront
    double co[NA], eo[NA], acc[NA];
    size_t so[NA];
#pragma unroll
    for (int l = 0; l < NB; ++l) {
        const bool ok = l < nb;
        const int s = ok ? l0 + l : l0;
        co[l] = ok ? cf[(size_t)s * NC + vc] : 0.0;
        eo[l] = ok && !PLAIN ? ec[(size_t)s * NC + vc] : 0.0;
        so[l] = (size_t)s * ss;
        acc[l] = 0.0;
    }
    const double wz = PLAIN ? 0.0 : sig[(size_t)i * NC + vc], wu = PLAIN ? 0.0 : cu[vc],
                 wr = PLAIN ? 0.0 : cr[vc];
    double *U = basis + (size_t)i * ss, *UN = U + ss;
    double accr = 0.0, accu = 0.0;
    int buf = 0;
    for (int64_t r = r0; r < r1; r += R) {
        double u[R], z[R], q[R][NA];
        size_t e[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            e[j] = (size_t)min(r + j, r1 - 1) * C + c;
            u[j] = U[e[j]];
            z[j] = PLAIN ? 0.0 : Z[e[j]];
        }
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int l = 0; l < NB; ++l) q[j][l] = __builtin_nontemporal_load(basis + so[l] + e[j]);
        __builtin_amdgcn_sched_barrier(0);
        double rr[R], un[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            double a = 0.0, b = 0.0;
#pragma unroll
            for (int l = 0; l < NB; ++l) {
                a += co[l] * q[j][l];
                if (!PLAIN) b += eo[l] * q[j][l];
            }
            rr[j] = a;
            un[j] = b;
        }
        if (W > 1) {
            double2 *x = xch + (size_t)buf * W * R * 64;
#pragma unroll
            for (int j = 0; j < R; ++j) x[(w * R + j) * 64 + lane] = make_double2(rr[j], un[j]);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < R; ++j) {
                double a = 0.0, b = 0.0;
                for (int q2 = 0; q2 < W; ++q2) {
                    const double2 p = x[(q2 * R + j) * 64 + lane];
                    a += p.x;
                    b += p.y;
                }
                rr[j] = a;
                un[j] = b;
            }
            buf ^= 1;
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const bool live = r + j < r1;
            const double rv = u[j] - rr[j];
            double uv = rv;
            if (!PLAIN) {
                uv = wz * z[j] - wu * u[j] - un[j];
                uv -= wr * rv;
            }
            if (w == 0 && live && colok) {
                if (!PLAIN || store_u) U[e[j]] = rv;
                if (!PLAIN && store_u) UN[e[j]] = uv;
            }
            uv = live ? uv : 0.0;
#pragma unroll
            for (int l = 0; l < NB; ++l) acc[l] += q[j][l] * uv;
            accr += rv * uv;
            accu += uv * uv;
        }
    }
    if (!colok) return;
    double *P = part + (size_t)chunk * rows * C + c;
#pragma unroll
    for (int l = 0; l < NB; ++l)
        if (l < nb) P[(size_t)(1 + l0 + l) * C] = acc[l];
    if (w == 0) {
        P[0] = accu;
        if (!PLAIN) P[(size_t)(1 + i) * C] = accr;
    }
}

// ------------------------------------------------------------------ launchers

void launch_dot_uz(const Plan &p, int i, const void *z, hipStream_t st)
{
    const unsigned grid = (unsigned)((int64_t)p.nchunk * p.nct);
    const double *u = (const double *)p.basis + (size_t)i * slot_elems(p);
    if (i == 0) {
        k_uz_scale<<<(p.nseg * p.C + 63) / 64, 64 * kFinWaves, 0, st>>>(p.C, p.nseg, p.part_rows, p.seg_chunk,
                                                                        p.part, p.kappa);
        k_dot_uz<true><<<grid, 256, 0, st>>>(p.C, p.nct, p.rpc, p.nseg, p.seg_row, p.seg_chunk, u,
                                             (const double *)z, p.kappa, p.part_rows, 1, p.part);
    } else {
        k_dot_uz<false><<<grid, 256, 0, st>>>(p.C, p.nct, p.rpc, p.nseg, p.seg_row, p.seg_chunk, u,
                                              (const double *)z, p.kappa, p.part_rows, i + 1, p.part);
    }
}

// Chunk sums of the first `rows` rows.
static void sweep_sum(const Plan &p, int rows, hipStream_t st)
{
    k_sweep_sum<<<dim3((p.nseg * p.C + 63) / 64, rows), 64 * kFinWaves, 0, st>>>(p.C, p.nseg, p.part_rows,
                                                                               p.seg_chunk, p.part);
}

void launch_sweep_fin(const Plan &p, int i, hipStream_t st)
{
    sweep_sum(p, i == 0 ? 3 : (i < p.k ? i + 2 : i + 1), st);
    const size_t lds = sizeof(double) * 64 * ((size_t)i + 16);
    if (lds > (size_t)64 << 10)   // more than the default of dynamic LDS (not a stream operation)
        (void)hipFuncSetAttribute((const void *)k_sweep_fin, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k_sweep_fin<<<(p.nseg * p.C + 63) / 64, 512, lds, st>>>(
        p.C, p.nseg, p.part_rows, i, p.k, DBL_EPSILON, p.seg_chunk, p.part, p.kappa, p.nu, p.sig, p.alpha, p.beta,
        p.cf, p.ec, p.cu, p.cr, p.runmax, p.active, p.kused, p.Ct, p.c_off);
}

void launch_arn_sweep_fin(const Plan &p, int i, hipStream_t st)
{
    sweep_sum(p, i + 1, st);
    k_arn_sweep_fin<<<(p.nseg * p.C + 63) / 64, 512, 0, st>>>(
        p.C, p.nseg, p.part_rows, i, p.k, DBL_EPSILON, p.seg_chunk, p.part, p.nu, p.sig, p.H, p.cf, p.ec, p.cu,
        p.cr, p.runmax, p.active, p.kused, p.Ct, p.c_off);
}

void launch_arn_dots_fin(const Plan &p, int i, hipStream_t st)
{
    const int NC = p.nseg * p.C;
    k_arn_dots_fin<<<dim3((NC + 63) / 64, i + 1), 64 * kFinWaves, 0, st>>>(
        p.C, p.nseg, p.part_rows, i, p.k, p.seg_chunk, p.part, p.sig, p.active, p.cf, p.H);
}

template <int NB, bool PLAIN, int WMAX = 4>
static void sweep_t(const Plan &p, int i, int W, const void *z, bool store, hipStream_t st)
{
    constexpr int R = NB > 20 ? 1 : (NB > 8 ? 2 : 4);
    k_sweep<NB, R, PLAIN, WMAX><<<(unsigned)((int64_t)p.nchunk * p.nct), 64 * W,
                            W > 1 ? sizeof(double2) * 2 * W * R * 64 : 0, st>>>(
        p.C, p.nct, p.rpc, p.nseg, p.seg_row, p.seg_chunk, (double *)p.basis, slot_elems(p), i,
        (const double *)z, p.sig, p.cf, p.ec, p.cu, p.cr, store ? 1 : 0, p.part_rows, p.part);
}

template <bool PLAIN>
static void sweep_nb(const Plan &p, int i, const void *z, bool store, hipStream_t st)
{
    // As few wavefronts as hold the slots: with one there is no exchange, and the rows
    // of a step of R are fewer as the slots are more (28 slots, one row: 254
    // registers).  At most 16 slots and seven wavefronts took, against 28 and four:
    // 64^3 x 512, k = 30 119.6 ms of sweeps, 116.3; 32^3 x 64, k = 100 19.7, 18.5;
    // Arnoldi 40^3 x 128, k = 30 14.3, 13.8; 24 and 30 slots are no faster.
    const int W = i > kSweepSlots ? (i + kSweepSlots - 1) / kSweepSlots : 1;
    const int nb = (i + W - 1) / W;
    if constexpr (!PLAIN) {
        if (W > 4) {   // 113 to 127 slots: 23 to 26 in each of five wavefronts (at most 256 registers)
            switch (nb) {
#define ECNT_CASE(N)                                 \
    case N:                                          \
        sweep_t<N, false, 5>(p, i, W, z, store, st); \
        return;
                ECNT_CASE(23) ECNT_CASE(24) ECNT_CASE(25) ECNT_CASE(26)
#undef ECNT_CASE
            }
        }
    }
    switch (nb) {
#define ECNT_CASE(N)                               \
    case N:                                        \
        sweep_t<N, PLAIN>(p, i, W, z, store, st);  \
        break;
        ECNT_CASE(0) ECNT_CASE(1) ECNT_CASE(2) ECNT_CASE(3) ECNT_CASE(4) ECNT_CASE(5)
        ECNT_CASE(6) ECNT_CASE(7) ECNT_CASE(8) ECNT_CASE(9) ECNT_CASE(10) ECNT_CASE(11)
        ECNT_CASE(12) ECNT_CASE(13) ECNT_CASE(14) ECNT_CASE(15) ECNT_CASE(16) ECNT_CASE(17)
        ECNT_CASE(18) ECNT_CASE(19) ECNT_CASE(20) ECNT_CASE(21) ECNT_CASE(22) ECNT_CASE(23)
        ECNT_CASE(24) ECNT_CASE(25) ECNT_CASE(26) ECNT_CASE(27) ECNT_CASE(28)
#undef ECNT_CASE
    default:
        break;
    }
}

void launch_sweep(const Plan &p, int i, const void *z, bool store, hipStream_t st)
{
    sweep_nb<false>(p, i, z, store, st);
}

void launch_sweep_plain(const Plan &p, int i, bool store, hipStream_t st)
{
    sweep_nb<true>(p, i, nullptr, store, st);
}

}  // namespace ecnt

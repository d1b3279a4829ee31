// Factored absolute-value preconditioner of Section 6 on a block of columns:
//   M x   = |D|^{-1/2} L^{-1} P x      (gather, k_ldl_solve<FWD>, k_ldl_eapply)
//   M^* x = P^T L^{-T} |D|^{-1/2} x    (k_ldl_eapply, k_ldl_solve<BWD>, scatter)
// with P (A - tau I) P^T ~ L D L^T the factor of the columns' shift.
//
// The substitutions are sequential in the rows; the columns (probes) are the
// parallel dimension: one wavefront owns a column and walks the rows in
// column form, keeping the pending sums of the next kRing rows in registers,
// which serves any factor of bandwidth at most kRing.  The factor is used in
// band form (each row as 256 values by distance from the diagonal, built once
// per call), so no column indices are read.
//
// A few columns leave most of the chip idle, so the rows are also cut into P
// parts.  A part depends on the rows before it only through the pending sums
// s_p of its first rows (at most the bandwidth), and linearly:
//   s_{p+1} = S_p(b_p) - K_p s_p,
// S_p(b) the sums that part p leaves behind for right-hand side b when nothing
// comes in, K_p = S_p on the unit vectors (once per call and triangle).  A solve
// is then: every part with nothing coming in (for S_p(b_p) only), the chain of
// the s_p (small matrix-vector products), and every part again with its s_p,
// which is plain substitution.  The s_p of the chain carry its forward error,
// though, where plain substitution has only a residual of rounding; so there
// is one step of refinement: the sums that part p really leaves behind minus
// s_{p+1}, d_{p+1}, go through the same chain (e_{p+1} = d_{p+1} - K_p e_p) and
// every part adds its solution with right-hand side 0 and e_p coming in.  Y is
// stored and then added to, so the residual is a few roundings more than plain
// substitution's: componentwise 1.1e-16 to 9e-16 against 0.6e-16 to 2.8e-16 over
// factors with |K_p| up to 240, dropping none to 0.5 (1e-13 without the step).
// (Solving again from s_p + e_p does not do: a pass repeats its own rounding
// only for the same input, and that again is a forward error.)
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "ecount_internal.h"

namespace ecnt {

namespace {
constexpr int kRing = 256;   // band width (the largest bandwidth served)
// rows of padding before and after each band: a batch of rows staged past
// either end of the walk reads them (never used), so no row index is clamped
constexpr int kPad = 32;
}

// |D|^{-1/2} block by block, for one shift.  A 2 x 2 block [[a, b], [b, c]]
// (b != 0) has eigenvalues mu_{1,2} = (a + c)/2 +- r, r = hypot((a - c)/2, b),
// and f(D) = (f(mu_1) (D - mu_2 I) - f(mu_2) (D - mu_1 I)) / (mu_1 - mu_2) for
// f(mu) = |mu|^{-1/2} (Sylvester's formula).  With x = (a - c)/2,
// a - mu_2 = r + x = p, c - mu_2 = r - x = q (p, q >= 0, p q = b^2), so
//   f(D)_11 = (f1 p + f2 q) / 2r,  f(D)_22 = (f1 q + f2 p) / 2r,
//   f(D)_12 = (f1 - f2) b / 2r,
// the smaller of p, q taken as b^2 / the larger (no cancellation).
__global__ void k_ldl_eblocks(int64_t n, const double *__restrict__ dd,
                              const double *__restrict__ doff, double *__restrict__ ed,
                              double *__restrict__ eo)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (i > 0 && doff[i - 1] != 0.0) return;   // second row of a block: done by row i-1
    if (i + 1 < n && doff[i] != 0.0) {
        const double a = dd[i], b = doff[i], c = dd[i + 1];
        const double x = 0.5 * (a - c), r = hypot(x, b);
        const double big = r + fabs(x), small = (b * b) / big;
        const double p = x >= 0.0 ? big : small, q = x >= 0.0 ? small : big;
        const double mid = 0.5 * (a + c);
        const double f1 = 1.0 / sqrt(fabs(mid + r)), f2 = 1.0 / sqrt(fabs(mid - r));
        const double inv = 1.0 / (2.0 * r);
        ed[i] = (f1 * p + f2 * q) * inv;
        ed[i + 1] = (f1 * q + f2 * p) * inv;
        eo[i] = (f1 - f2) * b * inv;
        eo[i + 1] = 0.0;
    } else {
        ed[i] = 1.0 / sqrt(fabs(dd[i]));
        eo[i] = 0.0;
    }
}

// Y = |D|^{-1/2} (xs .* X) on columns [c_lo, c_hi): one thread per (row, column).
template <typename T>
__global__ __launch_bounds__(256) void k_ldl_eapply(int64_t n, int C, int c_lo, int c_hi,
                                                    const double *__restrict__ doff,
                                                    const double *__restrict__ ed,
                                                    const double *__restrict__ eo,
                                                    const T *__restrict__ X,
                                                    const double *__restrict__ xs,
                                                    T *__restrict__ Y)
{
    const int w = c_hi - c_lo;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n * w) return;
    const int64_t r = g / w;
    const int c = c_lo + (int)(g - r * w);
    const double sc = xs ? xs[c] : 1.0;
    auto x = [&](int64_t i) { return static_cast<double>(X[(size_t)i * C + c]) * sc; };
    double y;
    if (r + 1 < n && doff[r] != 0.0) y = ed[r] * x(r) + eo[r] * x(r + 1);
    else if (r > 0 && doff[r - 1] != 0.0) y = eo[r - 1] * x(r - 1) + ed[r] * x(r);
    else y = ed[r] * x(r);
    Y[(size_t)r * C + c] = static_cast<T>(y);
}

// Band form of one factor, built once per call: row i of L as 256 values
// bf[i][256 - d] = l_{i, i-d}, and row i of L^T as bb[i][256 - d] = l_{i+d, i}
// (d = 1..256; zeros where L has no entry), each with kPad zero rows before
// and after (bf and bb point at row 0).
__global__ void k_ldl_band_zero(int64_t n, double *__restrict__ bf, double *__restrict__ bb)
{
    const int64_t total = (n + 2 * kPad) * kRing;
    bf -= (size_t)kPad * kRing;
    bb -= (size_t)kPad * kRing;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
         g += (int64_t)gridDim.x * blockDim.x) {
        bf[g] = 0.0;
        bb[g] = 0.0;
    }
}

__global__ void k_ldl_band_fill(int64_t n, int64_t nnz, const int32_t *__restrict__ rp,
                                const int32_t *__restrict__ ci, const double *__restrict__ lv,
                                double *__restrict__ bf, double *__restrict__ bb)
{
    // a wavefront per row, its lanes over the row's entries (each entry has
    // its own slot in either band)
    const int64_t i = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= n) return;
    int64_t p0 = rp[i], p1 = rp[i + 1];
    p0 = p0 < 0 ? 0 : (p0 > nnz ? nnz : p0);
    p1 = p1 < p0 ? p0 : (p1 > nnz ? nnz : p1);
    for (int64_t p = p0 + lane; p < p1; p += 64) {
        const int64_t j = ci[p], d = i - j;
        if (j < 0 || j >= n || d < 1 || d > kRing) continue;   // outside the declared bandwidth
        bf[(size_t)i * kRing + kRing - d] = lv[p];
        bb[(size_t)j * kRing + kRing - d] = lv[p];
    }
}

// Y[r] = X[perm[r]] (gather) or Y[perm[r]] = X[r] (scatter) on columns [c_lo, c_hi).
template <typename T, bool GATHER>
__global__ __launch_bounds__(256) void k_ldl_permute(int64_t n, int C, int c_lo, int c_hi,
                                                     const int32_t *__restrict__ perm,
                                                     const T *__restrict__ X, T *__restrict__ Y)
{
    const int w = c_hi - c_lo;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n * w) return;
    const int64_t r = g / w;
    const int c = c_lo + (int)(g - r * w);
    int64_t pr = perm[r];
    pr = pr < 0 ? 0 : (pr >= n ? n - 1 : pr);
    if (GATHER) Y[(size_t)r * C + c] = X[(size_t)pr * C + c];
    else Y[(size_t)pr * C + c] = X[(size_t)r * C + c];
}

// Substitution with the unit triangular factor on columns [c_lo, c_hi), in
// column (right-looking) form:
//   FWD: y_r = X[r] - sum_{j<r} l_rj y_j, rows r = 0..n-1
//   BWD: w_r = X[r] - sum_{j>r} l_jr w_j, rows r = n-1..0
// (Y[r] = y_r / w_r).  In walk order t (FWD r = t, BWD r = n-1-t) the value of
// step t enters steps t+1 .. t+256 with the coefficients of one band row:
// band[r][256 - d] links step t to step t + d (FWD: column r of L, i.e. the
// band of L^T; BWD: row r of L).  A wavefront owns one column: lane q keeps
// the pending sums of steps T0 + q + 64 s (s = 0..4) of the current group of
// 64 steps in registers (5 slots: from step T0 + 63 the values reach
// T0 + 319).  Step t = T0 + Q0: lane Q0 forms y = X - pending, v_readlane
// broadcasts it through scalar registers, and every lane adds coefficient * y
// to its 5 pending sums; at the end of a group the sums shift by one slot.
// The chain from one row to the next is a subtraction, the broadcast and one
// FMA; the next step's 5 coefficients are read from LDS before the current
// step's broadcast (two register sets alternate by step parity).  Band rows
// are loaded 16 steps ahead into registers and staged into LDS per 16 steps
// between 64 zeros on each side (read for distances outside 1..256).  All
// shifts of the wave in one launch (each solve is a latency-bound chain, so
// the shifts' chains run side by side): blocks [blk0[s], blk0[s+1]) serve
// shift s, its columns [lo[s], hi[s]) and its factor's band.
struct LdlSolveSet {
    int nsh;
    int blk0[kMaxShifts + 1];
    int lo[kMaxShifts], hi[kMaxShifts];
    const double *band[kMaxShifts];
};

// A workgroup is four wavefronts on four columns of one part; they share the
// staged band rows (8 steps at a time in two buffers, one barrier per 8 steps;
// each wavefront loads and stages two of them), so the band is read once per
// four columns.  Three buffers, which let a step read the next batch's first
// coefficients ahead, measured the same.  A pass over 17 parts of 960 rows, 50
// columns, takes 61 to 67 us, about 66 ns a row.
//
// MODE 0: a whole solve in one part.
// MODE 1: the part with nothing carried in, for its carry out: part p's goes
//         to carry[p + 1]; part 0 stores Y as well (it is final).
// MODE 2: right-hand side e_j (j = 0..): the carry out is row j of K_p^T.
// MODE 3: starts from the sums carry[p], stores Y; what it carries out minus
//         carry[p + 1] goes to diff[p + 1] (not for the last part).
// MODE 4: right-hand side 0, starts from the corrections diff[p], adds to Y.
// Steps of part p: [p R, min(n, (p + 1) R)), R a multiple of 64.
template <typename T, bool FWD, int MODE>
__global__ __launch_bounds__(256) void k_ldl_solve(int64_t n, int C, int64_t R, int part0,
                                                   const LdlSolveSet set, const T *__restrict__ X,
                                                   T *__restrict__ Y, double *__restrict__ carry,
                                                   double *__restrict__ diff)
{
    int sh = 0;
    while (sh + 1 < set.nsh && (int)blockIdx.x >= set.blk0[sh + 1]) ++sh;
    const int c_lo = set.lo[sh], c_hi = set.hi[sh];
    const double *__restrict__ band = set.band[sh];
    const int blk = (int)blockIdx.x - set.blk0[sh];
    const int ncb = (c_hi - c_lo + 3) / 4;   // column blocks of the shift
    const int p = part0 + blk / ncb;
    constexpr int NS = 64;             // lanes per column, steps per group
    constexpr int NR = kRing / NS;     // the pending sums per lane are NR + 1
    constexpr int kBatch = 8;          // band rows staged at a time
    constexpr int kMine = kBatch / 4;  // of them by each wavefront
    constexpr int kRow = NS + kRing + NS;   // staged row: zeros, band, zeros
    __shared__ double stg[2][kBatch][kRow];
    const int q = threadIdx.x & 63, wv = uniform(threadIdx.x >> 6);
    const int craw = c_lo + (blk % ncb) * 4 + wv;
    const bool ok = craw < c_hi;
    const int c = ok ? craw : c_lo;
    const int64_t tb = p * R, te = tb + R < n ? tb + R : n;
#pragma unroll
    for (int u = 0; u < 2 * kMine; ++u) {
        double *z = stg[u / kMine][wv * kMine + u % kMine];
        z[q] = 0.0;
        z[NS + kRing + q] = 0.0;
    }

    auto row_of = [&](int64_t t) -> int64_t {
        const int64_t tt = t < n ? t : n - 1;   // past the end: repeat the last row (unused)
        return FWD ? tt : n - 1 - tt;
    };
    // Band rows of a batch in registers: values 2 q, 2 q + 1, 128 + 2 q, 129 + 2 q
    // of this wavefront's rows of steps t0 .. t0 + 7 (consecutive rows, up in
    // FWD, down in BWD); t0 < n + 24, so they stay within the kPad rows of
    // padding past either end.  Batches alternate between two register sets.
    double nvA[kMine][4], nvB[kMine][4];
    auto load_batch = [&](double (&nv)[kMine][4], int64_t t0) __attribute__((always_inline)) {
        const double2 *row0 =
            reinterpret_cast<const double2 *>(band + (FWD ? t0 : n - 1 - t0) * (int64_t)kRing);
#pragma unroll
        for (int u = 0; u < kMine; ++u) {
            const double2 *row = row0 + (FWD ? wv * kMine + u : -(wv * kMine + u)) * (kRing / 2);
            const double2 a = row[q], b = row[64 + q];
            nv[u][0] = a.x;
            nv[u][1] = a.y;
            nv[u][2] = b.x;
            nv[u][3] = b.y;
        }
    };
    auto stage_batch = [&](const double (&nv)[kMine][4], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kMine; ++u) {
            double2 *row = reinterpret_cast<double2 *>(stg[buf][wv * kMine + u] + NS);
            double2 a, b;
            a.x = nv[u][0];
            a.y = nv[u][1];
            b.x = nv[u][2];
            b.y = nv[u][3];
            row[q] = a;
            row[64 + q] = b;
        }
    };
    auto load_b = [&](int64_t t) -> T {
        if (MODE == 2) return T(t - tb == craw ? 1 : 0);
        if (MODE == 4) return T(0);
        return X[(size_t)row_of(t) * C + c];
    };

    double slot[NR + 1];
#pragma unroll
    for (int s2 = 0; s2 <= NR; ++s2) slot[s2] = 0.0;
    if (MODE == 3 || MODE == 4) {
        const double *in = (MODE == 3 ? carry : diff) + ((size_t)p * C + c) * kRing;
#pragma unroll
        for (int s2 = 0; s2 < NR; ++s2) slot[s2] = in[q + NS * s2];
    }
    T b_own = load_b(tb + q), b_next = load_b(tb + NS + q);

    // coefficients of a step (position Q0 in the group, staging row u) for
    // slot s: distance d = q - Q0 + 64 s, staged index 64 + 256 - d (zero
    // unless 1 <= d <= 256).  Lane q's slot 0 takes only zeros from step
    // T0 + q on, so its y is b - slot[0] at the end of the group.
    double ca[NR + 1], cb[NR + 1];
    auto coefs = [&](int Q0, int u, int buf, double (&c_)[NR + 1]) __attribute__((always_inline)) {
        const double *sr = stg[buf][u] + (NS - q + Q0);
#pragma unroll
        for (int s2 = 0; s2 <= NR; ++s2) c_[s2] = sr[NS * (NR - s2)];
    };
    // one step: Q0 = position in the group (compile-time), U = staging row
    auto step = [&]<int Q0>(std::integral_constant<int, Q0>, int u) __attribute__((always_inline)) {
        double(&cur)[NR + 1] = (Q0 & 1) ? cb : ca;
        double(&nxt)[NR + 1] = (Q0 & 1) ? ca : cb;
        if (u + 1 < kBatch) coefs(Q0 + 1, u + 1, (Q0 / kBatch) & 1, nxt);
        const double y = static_cast<double>(b_own) - slot[0];   // meaningful in lane Q0
        const int lo = __builtin_amdgcn_readlane(__double2loint(y), Q0);
        const int hi = __builtin_amdgcn_readlane(__double2hiint(y), Q0);
        const double yb = __hiloint2double(hi, lo);
#pragma unroll
        for (int s2 = 0; s2 <= NR; ++s2) slot[s2] += cur[s2] * yb;
        // every pending sum is complete after its step (the compiler would
        // otherwise defer the FMAs of slots 1.. to the end of the group and
        // hold every step's coefficients and y until then)
#pragma unroll
        for (int s2 = 1; s2 <= NR; ++s2) asm volatile("" : "+v"(slot[s2]));
    };
    // batch B of the group (steps 8 B .. 8 B + 7), staged in buffer B mod 2: the
    // next batch goes to the other buffer first, the one two later into the
    // registers that held that; FULL: the whole group lies before step te (no
    // test per step).  Every wavefront runs the same batches and barriers.
    auto batch = [&]<int B, bool FULL>(int64_t T0, std::integral_constant<int, B>,
                                       std::bool_constant<FULL>) __attribute__((always_inline)) {
        const int64_t tn = T0 + (B + 1) * kBatch;
        if (tn < te) {
            if constexpr (B & 1) {
                stage_batch(nvA, 0);
                load_batch(nvA, tn + 2 * kBatch);
            } else {
                stage_batch(nvB, 1);
                load_batch(nvB, tn + 2 * kBatch);
            }
        }
        coefs(B * kBatch, 0, B & 1, ca);
        [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
            ((FULL || T0 + B * kBatch + U < te ? step(std::integral_constant<int, B * kBatch + U>{}, U)
                                               : void()),
             ...);
        }(std::make_integer_sequence<int, kBatch>{});
        __syncthreads();
    };
    auto group = [&]<bool FULL>(int64_t T0, std::bool_constant<FULL> f) __attribute__((always_inline)) {
        batch(T0, std::integral_constant<int, 0>{}, f);
        batch(T0, std::integral_constant<int, 1>{}, f);
        batch(T0, std::integral_constant<int, 2>{}, f);
        batch(T0, std::integral_constant<int, 3>{}, f);
        batch(T0, std::integral_constant<int, 4>{}, f);
        batch(T0, std::integral_constant<int, 5>{}, f);
        batch(T0, std::integral_constant<int, 6>{}, f);
        batch(T0, std::integral_constant<int, 7>{}, f);
    };

    load_batch(nvA, tb);
    load_batch(nvB, tb + kBatch);
    stage_batch(nvA, 0);
    load_batch(nvA, tb + 2 * kBatch);
    __syncthreads();
    const bool store = ok && MODE != 2 && (MODE != 1 || p == 0);
    // after a group: store its y, shift the pending sums by one slot
    auto finish_group = [&](int64_t T0) __attribute__((always_inline)) {
        if (store && T0 + q < te) {
            T *y = Y + (size_t)row_of(T0 + q) * C + c;
            const double v = static_cast<double>(b_own) - slot[0];
            *y = static_cast<T>(MODE == 4 ? static_cast<double>(*y) + v : v);
        }
#pragma unroll
        for (int s2 = 0; s2 < NR; ++s2) slot[s2] = slot[s2 + 1];
        slot[NR] = 0.0;
        b_own = b_next;
        b_next = load_b(T0 + 2 * NS + q);
    };
    // the groups that end before step te, then the partial last group
    int64_t T0 = tb;
    for (; T0 + NS <= te; T0 += NS) {
        group(T0, std::true_type{});
        finish_group(T0);
    }
    if (T0 < te) {
        group(T0, std::false_type{});
        finish_group(T0);
    }
    if (MODE == 1 && ok) {
#pragma unroll
        for (int s2 = 0; s2 < NR; ++s2) carry[((size_t)(p + 1) * C + c) * kRing + q + NS * s2] = slot[s2];
    }
    if (MODE == 3 && ok && te < n) {
#pragma unroll
        for (int s2 = 0; s2 < NR; ++s2) {
            const size_t e = ((size_t)(p + 1) * C + c) * kRing + q + NS * s2;
            diff[e] = slot[s2] - carry[e];
        }
    }
    if (MODE == 2 && ok) {
        double *K = carry + ((size_t)(p - part0) * kRing + craw) * kRing;
#pragma unroll
        for (int s2 = 0; s2 < NR; ++s2) K[q + NS * s2] = slot[s2];
    }
}

// The chain of the carried sums, one workgroup per column, p = 1..P-2:
// v[p + 1] -= K_p v[p], from v[1] as it is, or from 0 with REFINE (s_1 is exact).
// K_p is stored by columns (K[p - 1][j][i]); a thread takes a quarter of the j for
// two i.  Bound: K_p's 512 KiB through one CU's L2 port, so the loads run ahead of
// the products by one batch and do not wait for the sums.
struct LdlChainSet {
    int nsh;
    int hi[kMaxShifts];
    const double *K[kMaxShifts];
};

template <bool REFINE>
__global__ __launch_bounds__(512) void k_ldl_chain(int C, int P, const LdlChainSet set,
                                                   double *__restrict__ carry)
{
    // a batch: 16 of the thread's 64 j, two of its i at once
    constexpr int KB = kRing, PARTS = 4, NJ = KB / PARTS, LB = 16, NB = NJ / LB;
    __shared__ double s[KB], red[PARTS][KB];
    const int c = blockIdx.x;
    int sh = 0;
    while (sh + 1 < set.nsh && c >= set.hi[sh]) ++sh;
    const int i2 = threadIdx.x & 127, part = threadIdx.x >> 7, j0 = part * NJ;
    const double2 *K = reinterpret_cast<const double2 *>(set.K[sh] + (size_t)j0 * KB) + i2;
    const size_t step = (size_t)C * kRing;
    double *cp = carry + step + (size_t)c * kRing;   // s_1
    if (threadIdx.x < KB) s[threadIdx.x] = REFINE ? 0.0 : cp[threadIdx.x];
    double2 v[LB], w[LB];
    const int total = (P - 2) * NB;
    auto load = [&](int b, double2 (&o)[LB]) {   // batch b of the flattened sequence
        const int bb = b < total ? b : total - 1;
        const double2 *src = K + (size_t)(bb / NB) * (KB * KB / 2) + (size_t)(bb % NB) * LB * (KB / 2);
#pragma unroll
        for (int j = 0; j < LB; ++j) o[j] = src[(size_t)j * (KB / 2)];
    };
    load(0, v);
    __syncthreads();
    double a0 = 0.0, a1 = 0.0;
    auto use = [&](int b, const double2 (&m)[LB]) {
        const double *sj = s + j0 + (b % NB) * LB;
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            a0 += m[j].x * sj[j];
            a1 += m[j].y * sj[j];
        }
    };
    for (int b = 0; b < total; b += NB) {
#pragma unroll
        for (int h = 0; h < NB; h += 2) {
            load(b + h + 1, w);
            use(h, v);
            load(b + h + 2, v);
            use(h + 1, w);
        }
        red[part][2 * i2] = a0;
        red[part][2 * i2 + 1] = a1;
        a0 = a1 = 0.0;
        __syncthreads();
        if (threadIdx.x < KB) {
            const int i = threadIdx.x;
            const size_t nx = (size_t)(b / NB + 1) * step + i;
            const double t = cp[nx] - ((red[0][i] + red[1][i]) + (red[2][i] + red[3][i]));
            s[i] = t;
            cp[nx] = t;
        }
        __syncthreads();
    }
}

static double ldl_row_cycles(double wavefronts)
{
    const double issue = 60.0 / 1024.0 * wavefronts;
    return issue > 190.0 ? issue : 190.0;
}

int64_t ldl_part_rows(int64_t n, int P) { return ((n + P - 1) / P + 63) / 64 * 64; }

// Parts of the rows: the count with the least estimated time of a solve, in
// cycles (64-bit vectors only: the 32-bit form rounds each y once).  A step of
// the walk takes about 190 cycles, or 60 of issue per wavefront on a SIMD; a
// chain step 12500 (512 KiB through one CU's port: 5.0 us); K_p costs 256 more
// columns per part and triangle once per call, spread over 2 k solves.  n =
// 16129, 50 columns, k = 6: 17 parts of 960 rows, 343 us a solve (three passes of
// 64 us, two chains of 75), against 1140 us whole; below about 2500 rows, or with
// a thousand columns, it stays whole.
void ldl_plan_parts(Plan &p)
{
    p.ldl_parts = 1;
    if (p.prec_kind != 3 || p.vec_f32) return;
    const double cols = p.wave_cols, whole = p.n * ldl_row_cycles(cols);
    double best = 0.8 * whole;
    for (int P = 4; P <= 64; ++P) {   // (three walks of n / P rows: fewer parts gain nothing)
        const int64_t R = ldl_part_rows(p.n, P);
        if (R < kRing || (P - 1) * R >= p.n) continue;
        const double setup = R * ldl_row_cycles((double)kRing * (P - 2)) * p.S / p.k;
        const double t = 3.0 * R * ldl_row_cycles(cols * P) + 2.0 * (P - 2) * 12500.0 +
                         40000.0 + setup;
        if (t < best) {
            best = t;
            p.ldl_parts = P;
        }
    }
}

size_t ldl_chain_doubles(const Plan &p)   // K of both triangles of every shift
{
    return p.ldl_parts > 1 ? (size_t)2 * p.S * (p.ldl_parts - 2) * kRing * kRing : 0;
}

size_t ldl_carry_doubles(const Plan &p)
{
    return p.ldl_parts > 1 ? (size_t)2 * p.ldl_parts * p.wave_cols * kRing : 0;
}

int ldl_ring_rows() { return kRing; }

size_t ldl_band_bytes(int64_t n, int S) { return sizeof(double) * 2 * (size_t)S * (n + 2 * kPad) * kRing; }

// row 0 of the band of shift s: which = 0 rows of L, 1 rows of L^T
static double *band_of(const Plan &p, int s, int which)
{
    return p.band + ((size_t)(2 * s + which) * (p.n + 2 * kPad) + kPad) * kRing;
}

// K_1..K_{P-2} of shift s: which = 0 forward (L), 1 back substitution
static double *chain_of(const Plan &p, int s, int which)
{
    return p.ldl_chain + (size_t)(2 * s + which) * (p.ldl_parts - 2) * kRing * kRing;
}

void launch_ldl_eblocks(const Plan &p, hipStream_t st)
{
    for (int s = 0; s < p.S; ++s) {
        double *ed = p.e_blk + (size_t)s * 2 * p.n, *eo = ed + p.n;
        k_ldl_eblocks<<<(unsigned)((p.n + 255) / 256), 256, 0, st>>>(p.n, p.ldl[s].dd, p.ldl[s].doff,
                                                                     ed, eo);
        double *bf = band_of(p, s, 0), *bb = band_of(p, s, 1);
        k_ldl_band_zero<<<1024, 256, 0, st>>>(p.n, bf, bb);
        k_ldl_band_fill<<<(unsigned)((p.n + 3) / 4), 256, 0, st>>>(
            p.n, p.ldl[s].nnz, p.ldl[s].lrp, p.ldl[s].lci, p.ldl[s].lval, bf, bb);
    }
    if (p.ldl_parts == 1) return;
    // K_p, p = 1..P-2, of both triangles: a shift at a time (each fills the chip)
    for (int s = 0; s < p.S; ++s) {
        LdlSolveSet set;
        set.nsh = 1;
        set.lo[0] = 0;
        set.hi[0] = kRing;
        set.blk0[0] = 0;
        set.blk0[1] = (p.ldl_parts - 2) * (kRing / 4);
        const int64_t R = ldl_part_rows(p.n, p.ldl_parts);
        set.band[0] = band_of(p, s, 1);
        k_ldl_solve<double, true, 2><<<set.blk0[1], 256, 0, st>>>(p.n, p.C, R, 1, set, nullptr, nullptr,
                                                                  chain_of(p, s, 0), nullptr);
        set.band[0] = band_of(p, s, 0);
        k_ldl_solve<double, false, 2><<<set.blk0[1], 256, 0, st>>>(p.n, p.C, R, 1, set, nullptr, nullptr,
                                                                   chain_of(p, s, 1), nullptr);
    }
}

// columns of the wave that belong to shift s: [lo, hi)
static inline bool shift_cols(const Plan &p, int s, int &lo, int &hi)
{
    const int g0 = s * p.m, g1 = (s + 1) * p.m;
    lo = (g0 > p.c_off ? g0 : p.c_off) - p.c_off;
    hi = (g1 < p.c_off + p.C ? g1 : p.c_off + p.C) - p.c_off;
    return hi > lo;
}

template <typename T>
static void ldl_t(const Plan &p, int what, const void *X, const double *xs, void *Y, hipStream_t st)
{
    if (what == 1 || what == 2) {
        // forward substitution walks the columns of L (the band of L^T),
        // back substitution the rows of L
        LdlSolveSet set;
        LdlChainSet ch;
        set.nsh = 0;
        for (int s = 0; s < p.S; ++s) {
            int lo, hi;
            if (!shift_cols(p, s, lo, hi)) continue;
            const double *bf = band_of(p, s, 0), *bb = band_of(p, s, 1);
            const int k = set.nsh++;
            set.lo[k] = lo;
            set.hi[k] = hi;
            set.band[k] = what == 1 ? bb : bf;
            ch.hi[k] = hi;
            ch.K[k] = p.ldl_parts > 1 ? chain_of(p, s, what == 1 ? 0 : 1) : nullptr;
        }
        ch.nsh = set.nsh;
        if (set.nsh == 0) return;
        const int P = p.ldl_parts;
        const int64_t R = P > 1 ? ldl_part_rows(p.n, P) : (p.n + 63) / 64 * 64;
        auto blocks = [&](int parts) {   // a block per part and four columns of a shift
            set.blk0[0] = 0;
            for (int k = 0; k < set.nsh; ++k)
                set.blk0[k + 1] = set.blk0[k] + parts * ((set.hi[k] - set.lo[k] + 3) / 4);
            return (unsigned)set.blk0[set.nsh];
        };
        double *diff = p.ldl_carry + (P > 1 ? (size_t)P * p.C * kRing : 0);
        auto solve = [&](auto mode, int part0, int parts) {
            const unsigned grid = blocks(parts);
            if (what == 1)
                k_ldl_solve<T, true, decltype(mode)::value><<<grid, 256, 0, st>>>(
                    p.n, p.C, R, part0, set, (const T *)X, (T *)Y, p.ldl_carry, diff);
            else
                k_ldl_solve<T, false, decltype(mode)::value><<<grid, 256, 0, st>>>(
                    p.n, p.C, R, part0, set, (const T *)X, (T *)Y, p.ldl_carry, diff);
        };
        if (P == 1) {
            solve(std::integral_constant<int, 0>{}, 0, 1);
            return;
        }
        solve(std::integral_constant<int, 1>{}, 0, P - 1);
        k_ldl_chain<false><<<p.C, 512, 0, st>>>(p.C, P, ch, p.ldl_carry);
        solve(std::integral_constant<int, 3>{}, 1, P - 1);
        k_ldl_chain<true><<<p.C, 512, 0, st>>>(p.C, P, ch, diff);
        solve(std::integral_constant<int, 4>{}, 2, P - 2);
        return;
    }
    for (int s = 0; s < p.S; ++s) {
        int lo, hi;
        if (!shift_cols(p, s, lo, hi)) continue;
        const LdlDev &f = p.ldl[s];
        const double *ed = p.e_blk + (size_t)s * 2 * p.n, *eo = ed + p.n;
        const int64_t total = p.n * (hi - lo);
        const unsigned egrid = (unsigned)((total + 255) / 256);
        switch (what) {
        case 0:
            k_ldl_eapply<T><<<egrid, 256, 0, st>>>(p.n, p.C, lo, hi, f.doff, ed, eo, (const T *)X,
                                                   xs, (T *)Y);
            break;
        case 3:
            k_ldl_permute<T, true><<<egrid, 256, 0, st>>>(p.n, p.C, lo, hi, f.perm, (const T *)X,
                                                          (T *)Y);
            break;
        case 4:
            k_ldl_permute<T, false><<<egrid, 256, 0, st>>>(p.n, p.C, lo, hi, f.perm, (const T *)X,
                                                           (T *)Y);
            break;
        default:
            break;
        }
    }
}

// what: 0 = |D|^{-1/2} blocks (with the column scales xs), 1 = forward
// substitution with L, 2 = back substitution with L^T, 3 = gather by P,
// 4 = scatter by P^T
void launch_ldl(const Plan &p, int what, const void *X, const double *xs, void *Y, hipStream_t st)
{
    if (p.vec_f32) ldl_t<float>(p, what, X, xs, Y, st);
    else ldl_t<double>(p, what, X, xs, Y, st);
}

}  // namespace ecnt

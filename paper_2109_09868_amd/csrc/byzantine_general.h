// The locators in their general form, any nodes and up to 64 available workers: the full system of a class in LDS, a lane to
// a column.
#pragma once

#include "byzantine_common.h"

namespace approxifer {

// Rank of |a_r| among the n rows of one class (LDS key[n]); the A smallest vote for their worker.
// Called by the lanes of one class, lane j of `width` handling rows j, j+width, ..
__device__ __forceinline__ void pick_and_vote(const double *key, const int *avail, int n, int A, int j, int width,
                                              int *votes) {
    for (int r = j; r < n; r += width) {
        const double mine = key[r];
        int rank = 0;                                  // equal magnitudes keep ascending worker order
        for (int o = 0; o < n; ++o) {
            const double other = key[o];
            rank += (other < mine || (other == mine && o < r)) ? 1 : 0;
        }
        if (rank < A) atomicAdd(&votes[avail[r]], 1);
    }
}

// Householder reflector of a pivot column x (rows k..): returns alpha = -sign(x_k) ||x|| and the factor
// f = 2 v^T a / (v^T v) for a column a, v = x - alpha e_k, given sigma = x^T x, d = x^T a.
struct Reflector {
    double alpha, f;
    bool degenerate;
};
__device__ __forceinline__ Reflector reflector(double sigma, double d, double xkk, double akj) {
    Reflector h;
    h.degenerate = !(sigma > 0.0);
    // a zero (or NaN) column: the caller applies no reflection; alpha and f stay finite so that a factor 0 times
    // them is 0 and not NaN (an exactly singular system must keep its exact zero on the diagonal)
    const double s = h.degenerate ? 1.0 : sigma;
    const double nrm = sqrt_normal(s);
    h.alpha = (xkk >= 0.0) ? -nrm : nrm;
    const double scale = rcp_normal(fma(-h.alpha, xkk, s));   // 2 / (v^T v) = 1 / (sigma + |x_k| ||x||)
    h.f = scale * fma(-h.alpha, akj, d);
    return h;
}

constexpr int kInverseRounds = 24;      // inverse-iteration rounds before a class goes to the Jacobi iteration
constexpr int kJacobiSweeps = 30;

// Algorithm 1's fit needs a null vector of the homogeneous system: the right singular vector of the smallest
// singular value of its triangular factor R (rows 0..W2-1 of mat, row stride LD, lane j owns row j).  Writes the Q
// half of that vector to coef[0..M-1] (coefficients of columns M..W2-1); its length and sign are immaterial.
//
//  1. Inverse iteration z <- (R^T R)^-1 z, two triangular solves per round.  When the data are rational up to
//     rounding -- the case the locator is built for -- the smallest singular value is orders of magnitude below the
//     next and two to four rounds settle z: successive iterates within 1e-11, or no longer approaching each other.
//     A steady slow decay (two close smallest singular values) is extrapolated to its limit, Aitken's way.
//  2. Classes that have not settled after kInverseRounds (no gap: data that fit no rational function; or a zero on
//     the diagonal) get the full answer from one-sided Jacobi on G = R^T: lane j owns column j of G, which is row j
//     of mat; a step rotates W2/2 disjoint pairs of columns (round-robin pairing, W2 - 1 steps per sweep) until all
//     are orthogonal to rounding; the columns then are sigma_i v_i, v_i the right singular vectors of R, and the
//     shortest is the one wanted.  Both lanes of a pair read both columns and write their own: the new value of
//     element t depends on both reads of element t, and the lanes of a wave run in lock step, so no lane sees a
//     half-rotated pair.
// jacobi_only (wave-uniform): the caller's own inverse iteration has already failed to settle; go to step 2.
__device__ __forceinline__ void homogeneous_q(double *mat, int LD, double *coef, double *key, int W2, int M, int j,
                                              bool live, bool jacobi_only = false) {
    double *own = mat + j * LD;
    // ---- 1. inverse iteration; R mirrored into the lower triangle so that both solves read rows ----------------
    double colsq = 0.0;                                   // |column j of R|^2 = |column j of the system|^2
    for (int t = 0; t <= j; ++t) colsq = fma(mat[t * LD + j], mat[t * LD + j], colsq);
    if (live) {
        for (int t = 0; t < j; ++t) own[t] = mat[t * LD + j];
        // An exactly singular system (K = 1: the good workers return one and the same number) leaves a zero on the
        // diagonal.  Its null vector is the answer, but a zero pivot stops the solves and, in the Jacobi fallback, a
        // zero singular value wipes out its own vector (the columns there are sigma_i v_i).  A pivot below 1e-24 of
        // its column is raised to that: the null vector moves by 1e-24, far below the rounding of everything else.
        const double floor = 1e-24 * sqrt(colsq);
        if (fabs(own[j]) < floor) own[j] = own[j] < 0.0 ? -floor : floor;
    }
    __builtin_amdgcn_wave_barrier();
    const double rd = 1.0 / own[j];                     // still zero (a zero column): nothing settles, nor matters
    double z = 1.0 + 0.25 * (j % 3);
    double dd_prev = __builtin_inf();
    int since_jump = 0;
    bool settled = false;
    for (int round = jacobi_only ? kInverseRounds : 0; round < kInverseRounds; ++round) {
        double s = z;                                     // R^T w = z, forward
        for (int t = 0; t < W2; ++t) {
            const double rtj = mat[t * LD + j];           // issued ahead of the write -> read chain through key
            if (live && j == t) key[t] = s * rd;
            __builtin_amdgcn_wave_barrier();
            const double wt = key[t];
            if (j > t) s = fma(-rtj, wt, s);
        }
        __builtin_amdgcn_wave_barrier();
        s = key[j];                                       // R z' = w, backward
        for (int t = W2 - 1; t >= 0; --t) {
            const double rjt = mat[t * LD + j];           // the mirrored R[j][t]
            if (live && j == t) key[t] = s * rd;
            __builtin_amdgcn_wave_barrier();
            const double zt = key[t];
            if (j < t) s = fma(-rjt, zt, s);
        }
        __builtin_amdgcn_wave_barrier();
        double nn = 0.0;
        for (int t = 0; t < W2; ++t) nn = fma(key[t], key[t], nn);
        const double zn = key[j] * rcp_normal(sqrt_normal(nn));   // nn = 0, inf or NaN: NaN, and the class goes to Jacobi
        const double dz = zn - z;                         // z' . z > 0 always: no sign to align
        __builtin_amdgcn_wave_barrier();
        if (live) key[j] = dz * dz;
        __builtin_amdgcn_wave_barrier();
        double dd = 0.0;
        for (int t = 0; t < W2; ++t) dd += key[t];
        __builtin_amdgcn_wave_barrier();
        const double dd_before = dd_prev;
        // settled: the step is below 1e-11, or it has stopped shrinking at the level rounding allows (false for NaN)
        settled = settled || dd <= 1e-22 || (dd_prev <= 1e-16 && dd >= 0.25 * dd_prev);
        z = zn;
        dd_prev = dd;
        // Two close smallest singular values leave one slowly decaying error mode: z_k = v + r^k e.  Once the steps are
        // small and shrink by a steady factor r, jump to the limit of that sequence, z + r/(1-r) (z - z_previous); the
        // next two steps are no longer part of it, so at most every third round.
        ++since_jump;
        if (!settled && since_jump >= 3 && dd < 1e-4 && dd_before < __builtin_inf()) {
            const double r = sqrt(dd / dd_before);
            if (r > 0.05 && r < 0.97) {
                z = fma(r / (1.0 - r), dz, zn);
                since_jump = 0;
                dd_prev = __builtin_inf();
            }
        }
        if (__all((settled || !live) ? 1 : 0)) break;
    }
    if (live && settled && j >= M) coef[j - M] = z;
    const bool need = live && !settled;
    if (!__any(need ? 1 : 0)) {
        __builtin_amdgcn_wave_barrier();
        return;
    }

    // ---- 2. one-sided Jacobi for the classes that did not settle ----------------------------------------------
    if (need)
        for (int t = 0; t < j; ++t) own[t] = 0.0;
    __builtin_amdgcn_wave_barrier();
    const int m = W2 - 1;
    const double tol2 = (W2 * 2.220446049250313e-16) * (W2 * 2.220446049250313e-16);
    for (int sweep = 0; sweep < kJacobiSweeps; ++sweep) {
        bool rotated = false;
        for (int s = 0; s < m; ++s) {
            int k;                                        // this lane's partner: lane m plays s, the others mirror about s
            if (j == m) {
                k = s;
            } else if (j == s) {
                k = m;
            } else {
                k = 2 * s - j;
                if (k < 0) k += m;
                if (k >= m) k -= m;
            }
            const double *oth = mat + k * LD;
            double al = 0.0, be = 0.0, ga = 0.0;
            if (need) {
#pragma unroll 4
                for (int t = 0; t < W2; ++t) {
                    const double a = own[t], b = oth[t];
                    al = fma(a, a, al);
                    be = fma(b, b, be);
                    ga = fma(a, b, ga);
                }
            }
            const bool first = j < k;                     // the pair is (p, q), p < q; both lanes compute the same angle
            const double ap = first ? al : be, aq = first ? be : al;
            // rotate unless |g_p . g_q| <= tol |g_p| |g_q| (also skipped: NaN, and products that underflow to zero)
            const bool rot = need && ga * ga > tol2 * (ap * aq);
            if (rot) {
                // zeta = cot(2 phi), clamped so that its square stays finite (beyond 1e150 the rotation is the identity
                // to more digits than a double holds)
                const double zeta = fmin(fmax((aq - ap) * rcp_normal(2.0 * ga), -1e150), 1e150);
                const double tn = (zeta >= 0.0 ? 1.0 : -1.0) * rcp_normal(fabs(zeta) + sqrt_normal(fma(zeta, zeta, 1.0)));
                const double cs = rcp_normal(sqrt_normal(fma(tn, tn, 1.0)));
                const double so = first ? -cs * tn : cs * tn;      // g_p' = c g_p - s g_q,  g_q' = s g_p + c g_q
#pragma unroll 4
                for (int t = 0; t < W2; ++t) own[t] = fma(so, oth[t], cs * own[t]);
                rotated = true;
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (!__any(rotated ? 1 : 0)) break;
    }
    double nrm = 0.0;
    for (int t = 0; t < W2; ++t) nrm = fma(own[t], own[t], nrm);
    if (need) key[j] = (nrm == nrm) ? nrm : __builtin_inf();
    __builtin_amdgcn_wave_barrier();
    int jmin = 0;
    double best = key[0];
    for (int t = 1; t < W2; ++t) {
        const double v = key[t];
        if (v < best) {
            best = v;
            jmin = t;
        }
    }
    if (need && j >= M) coef[j - M] = mat[jmin * LD + j];
    __builtin_amdgcn_wave_barrier();                      // key is reused by the caller
}

// Algorithm 2, steps 1-2, for one class: row r of the n x 2M matrix  [x^0 .. x^(M-1) | -y x^1 .. -y x^(M-1) | y]
// (the last column is the right-hand side), written by lane j of the class's `width` lanes for rows j, j+width, ..
__device__ __forceinline__ void build_class_system(const float *__restrict__ pg, int64_t C, int64_t c, const int *avail,
                                                   const double *xs, int n, int M, double *mat, int LD, int j, int width,
                                                   bool live) {
    if (live) {
        for (int r = j; r < n; r += width) {
            const double x = xs[r];
            const double y = static_cast<double>(pg[static_cast<size_t>(avail[r]) * C + c]);
            double *row = mat + r * LD;
            double p = 1.0;
            for (int k = 0; k < M; ++k) {
                row[k] = p;                               // x^k
                if (k >= 1) row[M - 1 + k] = -y * p;      // -y x^k
                p *= x;
            }
            row[2 * M - 1] = y;
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// Householder QR in least-squares form, one lane per column: step k reflects column k onto e_k over rows k..n-1
// and applies the reflector to the columns right of it (and to the right-hand side).
__device__ __forceinline__ void factor_class_system(double *mat, int LD, int n, int j, int qr_steps, bool live) {
    for (int k = 0; k < qr_steps; ++k) {
        double sigma = 0.0, d = 0.0;
#pragma unroll 4
        for (int r = k; r < n; ++r) {
            const double vr = mat[r * LD + k];            // broadcast inside the class
            const double arj = mat[r * LD + j];
            sigma = fma(vr, vr, sigma);
            d = fma(vr, arj, d);
        }
        const double xkk = mat[k * LD + k];
        const double akj = mat[k * LD + j];
        const Reflector h = reflector(sigma, d, xkk, akj);
        __builtin_amdgcn_wave_barrier();
        if (live && !h.degenerate) {
            if (j > k) {
#pragma unroll 4
                for (int r = k; r < n; ++r) {
                    const double vr = (r == k) ? xkk - h.alpha : mat[r * LD + k];
                    mat[r * LD + j] = fma(-h.f, vr, mat[r * LD + j]);
                }
            } else if (j == k) {
                mat[k * LD + k] = h.alpha;                // R[k][k]
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Algorithm 2, steps 1-5, for the classes c0 .. c0+cpw-1 of one group, by one wave.
//   n        available workers (rows), M = K + A, W2 = 2M columns including the right-hand side
//   xs[n]    worker nodes of the available workers (LDS, shared by the workgroup)
//   scratch  this wave's LDS: per class  mat[n][W2] | coef[M] | key[n]
// Lane (cl, j) = (lane / W2, lane % W2) works on class c0 + cl; lanes beyond cpw classes idle.
// HOMOG: Algorithm 1's fit instead (Q_0 free).  The last column, y, then is one more column of the homogeneous
// system [V | -y x^1 .. -y x^(M-1) | y] whose coefficient is -Q_0; (P, Q) is its null vector of unit length.  jacobi_only: see
// homogeneous_q.
template <bool HOMOG>
__device__ __forceinline__ void locate_classes_wave(const float *__restrict__ pg, int64_t C, int64_t c0, int cpw,
                                                    const int *avail, const double *xs, int n, int M, int A,
                                                    double *scratch, int *votes, bool jacobi_only = false) {
    const int lane = lane_id();
    const int W2 = 2 * M;
    const int cols = W2 - 1;                 // unknowns P_0..P_{M-1}, Q_1..Q_{M-1}; column `cols` is the rhs
    const int cl = lane / W2;
    const int j = lane - cl * W2;
    const int64_t c = c0 + cl;
    const bool live = cl < cpw && c < C;     // this lane's class exists
    const int LD = HOMOG ? W2 + 1 : W2;     // row stride of mat; odd for the column rotations of Algorithm 1's fit
    const int per_class = n * LD + M + n;
    double *mat = scratch + (live ? cl : 0) * per_class;
    double *coef = mat + n * LD;
    double *key = coef + M;

    build_class_system(pg, C, c, avail, xs, n, M, mat, LD, j, W2, live);
    factor_class_system(mat, LD, n, j, HOMOG ? W2 : cols, live);

    if (HOMOG) {
        // ---- the null vector, then a_r = Q(x_r): Q_k = coef[k-1] for k >= 1, Q_0 = -coef[M-1] ----------------------
        homogeneous_q(mat, LD, coef, key, W2, M, j, live, jacobi_only);
        if (live) {
            for (int r = j; r < n; r += W2) {
                const double x = xs[r];
                double a = 0.0;
                for (int t = M - 2; t >= 0; --t) a = fma(a, x, coef[t]);
                a = fma(a, x, -coef[M - 1]);
                key[r] = (a != a) ? __builtin_inf() : fabs(a);
            }
        }
    } else {
        // ---- back substitution for Q_{M-1} .. Q_1 (unknowns cols-1 .. M); P is not needed ----
        // lane j holds the transformed right-hand side entry of row j.
        double s = (live && j < cols) ? mat[j * LD + cols] : 0.0;
        const double diag = (live && j < cols) ? mat[j * LD + j] : 1.0;
        for (int t = cols - 1; t >= M; --t) {
            if (live && j == t) coef[t - M] = s / diag;   // Q_{t-M+1}
            __builtin_amdgcn_wave_barrier();
            const double sol = coef[t - M];
            if (live && j < t) s = fma(-mat[j * LD + t], sol, s);
            __builtin_amdgcn_wave_barrier();
        }

        // ---- step 3: a_r = Q(x_r), Horner, one lane per row; steps 4-5: the A smallest |a_r| ----
        if (live) {
            for (int r = j; r < n; r += W2) {
                const double x = xs[r];
                double a = 0.0;
                for (int t = cols - 1; t >= M; --t) a = fma(a, x, coef[t - M]);
                a = fma(a, x, 1.0);                       // Q_0 = 1
                key[r] = (a != a) ? __builtin_inf() : fabs(a);
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    if (live) pick_and_vote(key, avail, n, A, j, W2, votes);
    __builtin_amdgcn_wave_barrier();
}

}  // namespace approxifer

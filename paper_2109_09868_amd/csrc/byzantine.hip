// ApproxIFER Byzantine decoder for gfx950: Algorithm 2 (error locator) followed by the decoder of
// Section 3, "ApproxIFER Decoding".
//
// Algorithm 2 fits, per class c, polynomials P (degree M-1) and Q (degree M-1, Q_0 = 1), M = K+A, to
//     P(x_r) - y_rc Q(x_r) = 0        over the n available workers (x_r their nodes),
// in the least-squares sense, reads a_r = Q(x_r), lets the A smallest |a_r| of every class vote and
// returns the A most voted workers.  The system is  V p + C_c q = y_c  with V the n x M Vandermonde
// matrix of the nodes and C_c = -diag(y_c) V[:, 1:].
//
// Four kernels compute the same thing:
//
//  * decode_byzantine_pairs_kernel (byzantine_pairs.h; the library's own worker nodes, a fixed number of at most four
//    missing, K+A <= 15, up to two workers more than eq. (3) asks for, three with K+A odd: pair_shape).  Two lanes to a class; no factorisation,
//    in the Chebyshev basis the projected system is sums of moments.
//
//  * decode_byzantine_proj_kernel (K+A <= 16, at most 48 available workers, n-M <= 32), one workgroup per
//    group.  V is the same for every class of a group, so its Householder QR is done ONCE per group,
//    by one wave with one lane per column of [V | I] held in registers (pivot columns travel by
//    v_readlane): that leaves U = the last n-M rows of Q^T, an orthonormal basis of range(V)'s
//    complement, in LDS.  Eliminating p exactly, class c only has to solve the (n-M) x (M-1) problem
//        min_q || U C_c q - U y_c ||,
//    so a class needs 16 lanes (lane = column, 15 = right-hand side), four classes share a wave, and
//    the systems are formed and solved entirely in registers, by modified Gram-Schmidt: what the other
//    lanes of the class need of a column reaches them inside the multiply-adds (see rows.h).
//    No LDS traffic and no barrier inside either factorisation.
//
//  * decode_byzantine_packed_kernel (the same for up to fifteen classes, see packed_domain): one to four
//    groups to a workgroup, factorised side by side, decoded by one matrix product each.
//
//  * decode_byzantine_general_kernel (everything else up to 64 available workers).  A class owns
//    2M neighbouring lanes, lane j owns COLUMN j of the full n x (2M-1) system, which sits in LDS
//    row-major; a Householder step walks down the pivot column (an LDS broadcast).
//
// All finish the same way: Q by back substitution, a_r = Q(x_r) by Horner's rule, the A smallest
// |a_r| (equal magnitudes: smaller worker index first; by counting ranks in the general kernel, by A
// rounds of a DPP minimum in the others) vote in an LDS histogram, the A most voted workers (equal
// counts: smaller index first) leave the available list, and the group is decoded over the rest.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "byzantine_common.h"
#include "byzantine_general.h"
#include "byzantine_pairs.h"
#include "rows.h"

// Built-in workspace of approxifer_decode_byzantine_static(): one copy per GPU the library runs on, held until
// the process ends.  In host code this name only stands for the symbol; its device address comes from
// hipGetSymbolAddress (see static_workspace below) and kernels receive that address as an argument.
static __device__ __align__(256) unsigned char scratch[APPROXIFER_STATIC_WORKSPACE_BYTES];

namespace approxifer {
namespace {

// ------------------------------------------------------------------------------------------------
// projected kernel: shared QR of the Vandermonde block, per-class QR in registers
// ------------------------------------------------------------------------------------------------
constexpr int kClsLanes = 16;      // lanes per class (one DPP row)
constexpr int kClsPerWave = 4;
constexpr int kPowers = 16;        // rows of the powers table: x^0 .. x^15
constexpr int kProjMaxM = 16;      // M - 1 <= 15 unknown columns in lanes 0..14, right-hand side in lane 15
// LDS layouts, all read a run of rows r at a time by lanes that differ in the other index: U[i][r] (rows padded to a
// multiple of four) and the powers Pw[e][r] = x_r^e with row stride lds_stride, the predictions Y[c][r] with y_stride.
// The strides keep runs 16-byte aligned and put the lanes of one 128-bit read into different banks.
constexpr int lds_stride(int NB) { return NB + 2; }                             // doubles: half of it is odd
constexpr int y_stride(int NB) { return (NB / 4) % 2 == 1 ? NB : NB + 4; }     // floats: a quarter of it is odd
// Register-array bound of Algorithm 1's locator for a tile of NB rows: eq. (3) gives M <= n / 2 <= NB / 2.
constexpr int hom_mt(int NB) { return NB / 2 < kProjMaxM ? NB / 2 : kProjMaxM; }
constexpr int ush_rows(int RM) { return (RM + 3) & ~3; }
constexpr int basis_stride(int NB) { return NB % 16 == 0 ? NB + 4 : NB; }      // of the basis kept in the workspace

// ---- once per group: U = rows M..n-1 of Q^T, V = Q R (one wave; lane = column of [V | I]) ----------
template <int K0, int NB>
struct SharedQrSteps {
    static __device__ __forceinline__ void run(double (&col)[NB], int lane, int M) {
        if (K0 < M) {
            double dt[2] = {0.0, 0.0};                       // two partial sums: shorter dependency chains
#pragma unroll
            for (int r = K0; r < NB; ++r) dt[(r - K0) & 1] = fma(read_lane(col[r], K0), col[r], dt[(r - K0) & 1]);
            const double d = dt[0] + dt[1];                  // x^T a for this lane's column a ..
            const double sigma = read_lane(d, K0);           // .. which in the pivot lane is x^T x
            const double xkk = read_lane(col[K0], K0);
            const Reflector h = reflector(sigma, d, xkk, col[K0]);
            // no branch: columns up to the pivot (and every column of a degenerate step) take the factor 0, so the
            // pivot values read for the dot products serve the update as well
            const double nf = (!h.degenerate && lane > K0) ? -h.f : 0.0;
            const double ckk = fma(nf, xkk - h.alpha, col[K0]);
            col[K0] = (!h.degenerate && lane == K0) ? h.alpha : ckk;      // R[k][k] in the pivot lane
#pragma unroll
            for (int r = K0 + 1; r < NB; ++r) col[r] = fma(nf, read_lane(col[r], K0), col[r]);
            SharedQrSteps<K0 + 1, NB>::run(col, lane, M);
        }
    }
};
template <int NB>
struct SharedQrSteps<kProjMaxM, NB> {
    static __device__ __forceinline__ void run(double (&)[NB], int, int) {}
};

// Pw[e][r] = x_r^e (LDS), n rows, M <= 16 columns.  Writes Ush[i][r] = U[i][r], i < RM, row stride lds_stride(NB).
// WITH_RANGE (Algorithm 1's locator needs the whole factorisation): also Q1sh[i][r] = row i < M of Q^T (16 rows of
// the same stride, rows from M on left as they are) and Rv[i][j] = R[i][j], the M x M triangular factor of V (row
// stride 16, zero below the diagonal).
template <int NB, int RM, bool WITH_RANGE = false>
__device__ __forceinline__ void shared_complement_basis(const double *Pw, int n, int M, double *Ush, double *Q1sh = nullptr,
                                                        double *Rv = nullptr) {
    const int lane = lane_id();
    double col[NB];
    const bool vandermonde = lane < M;                // lanes 0..M-1: V; lanes M..M+n-1: the identity
    const int e = vandermonde ? lane : 0;
#pragma unroll
    for (int r = 0; r < NB; ++r) {
        const double p = Pw[e * lds_stride(NB) + (r < n ? r : 0)];
        col[r] = (r < n) ? (vandermonde ? p : (lane - M == r ? 1.0 : 0.0)) : 0.0;
    }
    SharedQrSteps<0, NB>::run(col, lane, M);
    const int r_out = lane - M;                     // this lane holds column r_out of Q^T
    if (r_out >= 0 && r_out < n) {
#pragma unroll
        for (int row = 2; row < NB; ++row) {        // M >= 2 always
            const int i = row - M;
            if (i >= 0 && i < RM) Ush[i * lds_stride(NB) + r_out] = col[row];
        }
        if (WITH_RANGE) {
#pragma unroll
            for (int row = 0; row < kProjMaxM && row < NB; ++row)
                if (row < M) Q1sh[row * lds_stride(NB) + r_out] = col[row];
        }
    }
    if (WITH_RANGE && lane < M) {
#pragma unroll
        for (int row = 0; row < kProjMaxM && row < NB; ++row)
            if (row < M) Rv[row * kProjMaxM + lane] = row <= lane ? col[row] : 0.0;
    }
}

// ---- once per group, four groups to a wave: U = the last n - M columns of Q, transposed ----------------------------
// Householder reflectors of the group's Vandermonde block V (n x M) in the group's 16-lane row, lane = column, then
// the reflectors applied, last one first, to the unit vectors e_M .. e_(n-1), one per lane: Q e_(M+i) = H_0 .. H_(M-1)
// e_(M+i) is row i of U.  Every broadcast rides in a multiply-add (row_dot, row_axpy), so the wave factorises four
// groups in the issue slots that one took with the pivot column read lane by lane.
template <int K0, int NB, int MS>
struct RowReflectors {
    // lane K0 keeps v_K0 in rows K0.. of its column, 2 / v^T v in `sc` and R[K0][K0] in `diag`
    static __device__ __forceinline__ void factor(double (&a)[NB], int j, int M, double &sc, double &diag) {
        if constexpr (K0 < MS) {
            if (K0 < M) {
                double d0 = 0.0, d1 = 0.0;
                row_dot<K0, K0>(a, a, d0, d1);
                const double d = d0 + d1;                    // x^T a for this lane's column a ..
                const double sigma = row_bcast<K0>(d);       // .. which in the pivot lane is x^T x
                const double xkk = row_bcast<K0>(a[K0]);
                const bool zero = !(sigma > 0.0);            // no reflection (empty rows of the wave come here)
                const double sq = zero ? 1.0 : sigma;
                const double nrm = sqrt_normal(sq);
                const double alpha = xkk >= 0.0 ? -nrm : nrm;
                const double scale = zero ? 0.0 : rcp_normal(fma(-alpha, xkk, sq));
                const double nf = j > K0 ? -scale * fma(-alpha, a[K0], d) : 0.0;
                const double v0 = xkk - alpha;
                a[K0] = j == K0 ? v0 : fma(nf, v0, a[K0]);
                sc = j == K0 ? scale : sc;
                diag = j == K0 ? (zero ? xkk : alpha) : diag;
                row_axpy_self<K0, K0 + 1>(a, nf);            // lanes up to the pivot take the factor 0
                RowReflectors<K0 + 1, NB, MS>::factor(a, j, M, sc, diag);
            }
        }
    }
    static __device__ __forceinline__ void apply(const double (&a)[NB], double (&z)[NB], int M, double sc) {
        if constexpr (K0 < MS) {
            RowReflectors<K0 + 1, NB, MS>::apply(a, z, M, sc);
            if (K0 < M) {
                double d0 = 0.0, d1 = 0.0;
                row_dot<K0, K0>(a, z, d0, d1);
                const double nf = -row_bcast<K0>(sc) * (d0 + d1);
                row_axpy<K0, K0, NB>(z, a, nf);
            }
        }
    }
};

// One wave; lane row q works on group q: n_q workers avail_q[0..n_q), ascending (n_q = 0: none).  Pw[e][w] = x_w^e by
// worker, row stride `stride` as Ush.  Writes Ush_q[i * stride + w] = U[i][worker w] for i < n_q - M, and WITH_RANGE
// (Algorithm 1) Q1_q[i * stride + w], i < M, the same of the first M columns of Q, and Rv_q[16][16] the upper triangle of
// R; the rest of each is left as it is: zero.
template <int NB, bool WITH_RANGE>
__device__ __forceinline__ void rows_complement_basis(const double *Pw, const int *avail_q, int n, int M, double *Ush_q,
                                                      int stride, double *Q1_q, double *Rv_q) {
    constexpr int MS = NB / 2 < kProjMaxM ? NB / 2 : kProjMaxM;       // eq. (3): 2 M <= n <= NB
    const int j = lane_id() % kClsLanes;
    double a[NB], z[NB], sc = 0.0, diag = 0.0;
#pragma unroll
    for (int r = 0; r < NB; ++r) {
        const double p = Pw[j * stride + (r < n ? avail_q[r] : 0)];
        a[r] = (r < n && j < M) ? p : 0.0;
    }
    RowReflectors<0, NB, MS>::factor(a, j, M, sc, diag);
#pragma unroll
    for (int r = 0; r < NB; ++r) z[r] = r == M + j && r < n ? 1.0 : 0.0;
    RowReflectors<0, NB, MS>::apply(a, z, M, sc);
    if (M + j < n) {
#pragma unroll
        for (int r = 0; r < NB; ++r)
            if (r < n) Ush_q[j * stride + avail_q[r]] = z[r];
    }
    if (WITH_RANGE) {
#pragma unroll
        for (int r = 0; r < NB; ++r) z[r] = r == j && j < M && r < n ? 1.0 : 0.0;
        RowReflectors<0, NB, MS>::apply(a, z, M, sc);
        if (j < M && n > 0) {
#pragma unroll
            for (int r = 0; r < NB; ++r)
                if (r < n) Q1_q[j * stride + avail_q[r]] = z[r];
#pragma unroll
            for (int i = 0; i < MS; ++i)
                if (i <= j) Rv_q[i * kProjMaxM + j] = i == j ? diag : a[i];
        }
    }
}

// ---- per class: least squares of the projected system, in registers ------------------------------
// Modified Gram-Schmidt on [B | rhs] (lane = column): step K0 takes the part along column K0 out of every column,
//     nf_j = -(a_K0 . a_j) / (a_K0 . a_K0),    a_j += nf_j a_K0,
// and leaves a unit triangular system, nf being the negative of its row K0.  With the right-hand side carried as a
// column this is as backward stable for least squares as Householder reflections (it is Householder on [0; B], Bjorck
// 1967), takes no square root and no pivot reciprocals in the back substitution, and nothing has to be masked: columns
// up to the pivot are never read again.  It works on all RM rows at every step where reflections shrink, which the
// shorter scalar part more than pays for.  A zero column gives NaN, as dividing by a zero pivot does.
//   K = 12, A = 2 (28 x 14 tile), 8192 groups of 10 classes: 120 us a call with reflections, 91 us this way;
//   K = 8, A = 2 (20 x 10 tile), 2048 groups of 10 classes: 29.1 and 24.5 us.
// Steps K0 .. KEND-1 (those below `cols`).
template <int K0, int KEND, int RM>
struct ClassGramSchmidt {
    static __device__ __forceinline__ void run(double (&a)[RM], double (&nf)[KEND], int cols) {
        if (K0 < cols) {
            double d0 = 0.0, d1 = 0.0;
            row_dot<K0, 0>(a, a, d0, d1);
            const double d = d0 + d1;                        // x^T a for this lane's column a ..
            const double sigma = row_bcast<K0>(d);           // .. which in the pivot lane is x^T x
            nf[K0] = -d * rcp_normal(sigma);
            row_axpy_self<K0, 0>(a, nf[K0]);
            ClassGramSchmidt<K0 + 1, KEND, RM>::run(a, nf, cols);
        }
    }
};
template <int KEND, int RM>
struct ClassGramSchmidt<KEND, KEND, RM> {
    static __device__ __forceinline__ void run(double (&)[RM], double (&)[KEND], int) {}
};

// Solves the unit triangular system for the negative of its solution: nf[i] in lane t is minus entry (i, t), the
// negative of the right-hand side comes in in s and the negative of the solution leaves.
template <int T, int NS>
struct BackSubst {
    static __device__ __forceinline__ void run(const double (&nf)[NS], double (&s)[NS], int cols) {
        if (T < cols) {
            row_axpy<T, 0, T>(s, nf, s[T]);
        } else {
            s[T] = 0.0;                                   // no such unknown
        }
        BackSubst<T - 1, NS>::run(nf, s, cols);
    }
};
template <int NS>
struct BackSubst<-1, NS> {
    static __device__ __forceinline__ void run(const double (&)[NS], double (&)[NS], int) {}
};

// The same elimination for the triangular factor itself (Algorithm 1): r[K0] = row K0 of R in the lanes from K0 on.  A
// zero column leaves a zero row and takes nothing out of the others.
template <int K0, int KEND, int RM>
struct ClassTriangle {
    static __device__ __forceinline__ void run(double (&a)[RM], double (&r)[KEND], int cols) {
        if (K0 < cols) {
            double d0 = 0.0, d1 = 0.0;
            row_dot<K0, 0>(a, a, d0, d1);
            const double d = d0 + d1;                        // x^T a for this lane's column a ..
            const double sigma = row_bcast<K0>(d);           // .. which in the pivot lane is x^T x
            const double y = sigma > 0.0 ? rsqrt_normal(sigma) : 0.0;
            r[K0] = d * y;
            row_axpy_self<K0, 0>(a, -r[K0] * y);
            ClassTriangle<K0 + 1, KEND, RM>::run(a, r, cols);
        } else {
            r[K0] = 0.0;
            ClassTriangle<K0 + 1, KEND, RM>::run(a, r, cols);
        }
    }
};
template <int KEND, int RM>
struct ClassTriangle<KEND, KEND, RM> {
    static __device__ __forceinline__ void run(double (&)[RM], double (&)[KEND], int) {}
};

// The A smallest keys of a class (equal keys: smaller row first) vote.  Lane j of the class's 16-lane row holds the
// keys of rows j, j + 16, ..: |a_r|, infinity where it is not a number, NaN where there is no such row.  The minimum
// travels by itself (a NaN loses to any number); a ballot then finds the first row that has it.
template <int PR>
__device__ __forceinline__ void vote_smallest(double (&key)[PR], int A, bool live, const int *worker_of_row, int *votes) {
    const int lane = lane_id();
    const unsigned long long row_lanes = 0xffffull << (lane & 48);
    const unsigned long long before = row_lanes & ((1ull << lane) - 1ull);
    for (int pick = 0; pick < A; ++pick) {
        double m = key[0];
#pragma unroll
        for (int p = 1; p < PR; ++p) m = __builtin_fmin(m, key[p]);
        m = __builtin_fmin(m, dpp_exchange<kDppQuadXor1>(m));
        m = __builtin_fmin(m, dpp_exchange<kDppQuadXor2>(m));
        m = __builtin_fmin(m, dpp_exchange<kDppRowHalfMirror>(m));
        m = __builtin_fmin(m, dpp_exchange<kDppRowMirror>(m));
        bool open = true;                                 // no row of this class found yet
#pragma unroll
        for (int p = 0; p < PR; ++p) {
            const bool has = key[p] == m;
            const unsigned long long who = __ballot(has);
            if (open && has && (who & before) == 0ull) {
                const int r = lane % kClsLanes + p * kClsLanes;
                if (live) atomicAdd(&votes[worker_of_row != nullptr ? worker_of_row[r] : r], 1);
                key[p] = __builtin_nan("");
            }
            open = open && (who & row_lanes) == 0ull;
        }
    }
}

typedef double v2d __attribute__((ext_vector_type(2)));

// a[i] += sum_r U[i][r] y_r w_r over the NB rows r, this lane holding row i = lane % 16 of U (`u`), its class's
// predictions (`y`) and its column's powers (`w`): an outer product per row, whose factor U[i][r] reaches the lanes of
// the class inside the multiply-add.  On the vector ALUs on purpose: v_mfma_f64_16x16x4_f64 takes four classes' products
// in the same layout, but at 108 cycles each (measured; 16 % below the rate of plain multiply-adds) it holds the same
// issue slots and fills fourteen of sixteen columns: K = 12, A = 2, 28 workers, 8192 groups 71 us with it, 69 without;
// Algorithm 1 at K = 8, A = 2, 2048 groups 67 and 61 us.
template <int NB, int RM>
__device__ __forceinline__ void project_column(double (&a)[RM], const double *u, const float *y, const double *w) {
#pragma unroll
    for (int r = 0; r < NB; r += 4) {
        const v4f y4 = *reinterpret_cast<const v4f *>(y + r);
#pragma unroll
        for (int h = 0; h < 4; h += 2) {
            const v2d w2 = *reinterpret_cast<const v2d *>(w + r + h);
            const v2d u2 = *reinterpret_cast<const v2d *>(u + r + h);
            const double p0 = static_cast<double>(y4[h]) * w2[0], p1 = static_cast<double>(y4[h + 1]) * w2[1];
            constexpr int kLow = RM < kClsLanes ? RM : kClsLanes;
            row_outer<0, 0, kLow>(a, u2[0], p0);
            row_outer<0, 0, kLow>(a, u2[1], p1);
            if constexpr (RM > kClsLanes) {               // rows 16.. of U come from a second register of the lanes
                const v2d v2 = *reinterpret_cast<const v2d *>(u + kClsLanes * lds_stride(NB) + r + h);
                row_outer<kClsLanes, 0, RM - kClsLanes>(a, v2[0], p0);
                row_outer<kClsLanes, 0, RM - kClsLanes>(a, v2[1], p1);
            }
        }
    }
}

// Algorithm 2, steps 1-5, for four classes at a time, by one wave; lane / 16 is the class slot.  Per lane:
//   y[r] = the class's prediction of row r, float, zero where there is no answer (an empty slot points at zeros); `zeros`
//   the same number of zeros;  U: its group's U[i][r], zero where there is no such row or column;  live: the slot holds a
//   class;  bit r of rows: row r is an available worker;  votes: the counters of its group, by worker.
// Pw[e][r] = powers of the rows' nodes: the same rows for all four slots.  U and Pw in LDS, stride lds_stride(NB).
// A row is the r-th available worker, worker_of_row its index, or (worker_of_row null) the worker r itself.
template <int NB, int RM>
__device__ __forceinline__ void locate_classes_proj(const float *y, const float *zeros, const double *U, bool live,
                                                    unsigned long long rows, const int *worker_of_row, const double *Pw,
                                                    int M, int A, int *votes) {
    const int lane = lane_id();
    const int j = lane % kClsLanes;
    const int cols = M - 1;                               // unknowns Q_1 .. Q_{M-1}

    // the projected system B_c = U diag(y_c) [x^e]: column of this lane: y x^(j+1) for the unknown Q_(j+1), y for the
    // right-hand side, 0 on idle lanes (the signs of -y x^(j+1) q = y are left out: the solve below returns the negative)
    const int e = j < cols ? j + 1 : 0;
    double a[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) a[i] = 0.0;
    project_column<NB>(a, U + (j < RM ? j : 0) * lds_stride(NB), j < cols || j == kClsLanes - 1 ? y : zeros,
                       Pw + e * lds_stride(NB));

    constexpr int kSteps = RM - 1 < kProjMaxM - 1 ? RM - 1 : kProjMaxM - 1;   // most unknowns this tile can hold
    double nf[kSteps];
    ClassGramSchmidt<0, kSteps, RM>::run(a, nf, cols);

    double q[kSteps];                                     // minus the right-hand side in, Q_1 .. Q_{M-1} out
#pragma unroll
    for (int i = 0; i < kSteps; ++i) q[i] = row_bcast<kClsLanes - 1>(nf[i]);
    BackSubst<kSteps - 1, kSteps>::run(nf, q, cols);

    // a_r = Q(x_r) = 1 + sum_t q[t] x^(t+1) (q[t] = 0 for t >= cols), rows j, j+16, .. of this lane
    constexpr int PR = (NB + kClsLanes - 1) / kClsLanes;
    double key[PR];
#pragma unroll
    for (int p = 0; p < PR; ++p) {
        const int r = j + p * kClsLanes;
        const double x = Pw[lds_stride(NB) + (r < NB ? r : 0)];
        double av = 0.0;
#pragma unroll
        for (int t = kSteps - 1; t >= 0; --t) av = fma(av, x, q[t]);
        av = fma(av, x, 1.0);
        key[p] = ((rows >> r) & 1ull) ? (av == av ? fabs(av) : __builtin_inf()) : __builtin_nan("");
    }
    vote_smallest<PR>(key, A, live, worker_of_row, votes);
}

constexpr int kRegisterRounds = 64;     // .. and of the register form, whose rounds are cheap next to that fallback

// Sweeps over all entries (or back), f(i) and b(i) being this lane's multipliers of entry i.  Entries from M on are zero
// and take no branch: the multipliers that come from LDS are then read ahead of the chain.
template <int I, int MT>
struct TriangularSweeps {
    template <class F>
    static __device__ __forceinline__ void forward(double &s, F f) {
        row_sweep<I>(s, f(I));
        if constexpr (I + 1 < MT) TriangularSweeps<I + 1, MT>::forward(s, f);
    }
    template <class F, class B>
    static __device__ __forceinline__ void forward2(double &s, F f, double &t, B b) {
        row_sweep2<I>(s, f(I), t, b(I));
        if constexpr (I + 1 < MT) TriangularSweeps<I + 1, MT>::forward2(s, f, t, b);
    }
    template <class F>
    static __device__ __forceinline__ void backward(double &s, F f) {
        row_sweep<I>(s, f(I));
        if constexpr (I > 0) TriangularSweeps<I - 1, MT>::backward(s, f);
    }
    template <class F, class B>
    static __device__ __forceinline__ void backward2(double &s, F f, double &t, B b) {
        row_sweep2<I>(s, f(I), t, b(I));
        if constexpr (I > 0) TriangularSweeps<I - 1, MT>::backward2(s, f, t, b);
    }
};

// What the sweeps over R_V need, once per group, behind R_V itself: fv[i][j] = -R_V[i][j] / R_V[j][j] for i < j (the
// forward sweep of lane j), gv[k][j] = -R_V[j][k] / R_V[j][j] for k > j (its backward sweep), 1 / R_V[j][j].
constexpr int kVSquare = kProjMaxM * kProjMaxM;
constexpr int kVDoubles = 3 * kVSquare + kProjMaxM;      // R_V | fv | gv | reciprocal pivots
// Entry e of the squares (e < 256), by one thread each.  A pivot below 1e-24 of its column is raised to that.
__device__ __forceinline__ void sweep_multipliers(double *Rv, int e, int M) {
    const int i = e / kProjMaxM, j = e % kProjMaxM;
    double cs = 0.0;
    for (int t = 0; t < M; ++t) cs = fma(Rv[t * kProjMaxM + j], Rv[t * kProjMaxM + j], cs);
    double dv = Rv[j * kProjMaxM + j];
    const double least = 1e-24 * sqrt(cs);
    if (fabs(dv) < least) dv = dv < 0.0 ? -least : least;
    const double rdv = j < M ? 1.0 / dv : 0.0;
    Rv[kVSquare + e] = i < j ? -Rv[e] * rdv : 0.0;
    Rv[2 * kVSquare + e] = i > j && i < M ? -Rv[j * kProjMaxM + i] * rdv : 0.0;
    if (i == 0) Rv[3 * kVSquare + j] = rdv;
}

// Smallest right singular vector of the 2M x 2M factor R = [[R_V, B1], [0, R2]] of one class, by inverse iteration
// z <- (R^T R)^-1 z, entirely in the registers of the class's 16-lane row (lane j = index j of both halves of
// z = (p, q), M <= 15).  The four triangular solves of a round,
//     w1 = R_V^-T p,   w2 = R2^-T (q - B1^T w1),   q' = R2^-1 w2,   p' = R_V^-1 (w1 - B1 q'),
// are column sweeps: the entry that has just become final is broadcast along the row inside the multiply-add with which
// every lane takes its multiple; the division by the pivot is folded into the multipliers.  The two forward sweeps need
// the lane's COLUMN of R_V, B1, R2, the two backward ones its ROW: the columns of B1 and R2 and the row of B1 are held
// in registers, the row of R2 stays in the wave's LDS scratch through which it was transposed (T: 4 classes x MT x
// (MT + 1) doubles), R_V's multipliers are the group's (sweep_multipliers): with all of it in registers the 28-row tile
// spills (K = 12, A = 2, 8192 groups, a workgroup each: 427 us, 333 us this way).  Start vector, settling rule, extrapolation of a slowly decaying error mode and
// the floor under vanishing pivots are those of homogeneous_q (the LDS form, which stays the fallback for a class
// that has not settled after kRegisterRounds: it also holds the Jacobi iteration).
//   r2c[i] = R2[i][j] (i <= j), b1c[i] = B1[i][j]: this lane's columns; Rv: LDS, see kVDoubles.
//   MT >= M bounds the unrolling and the register arrays (the register tile of the kernel bounds M: M <= NB / 2).
// `live`: the row holds a class.  Returns q_j in `qv` and whether the class settled (the same value in all lanes of
// the row).
template <int MT>
__device__ __forceinline__ bool singular_vector_rows(const double (&r2c)[MT], const double (&b1c)[MT],
                                                     const double *Rv, double *T, int M, int j, int cl, bool live,
                                                     double &qv) {
    constexpr int LDT = MT + 1;
    const bool act = j < M;
    double *Tc = T + cl * MT * LDT;                        // M <= MT: lanes j >= MT hold no column and read no row
    // reciprocal pivot; one below 1e-24 of its column of R is raised to that (an exactly singular system keeps its null
    // vector to 1e-24, and the solves stay finite)
    double cs2 = 0.0, d2 = 0.0;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const double r2 = i < M && i <= j ? r2c[i] : 0.0;
        cs2 = fma(b1c[i], b1c[i], fma(r2, r2, cs2));
        d2 = i == j ? r2 : d2;
    }
    const double least = 1e-24 * sqrt(cs2);
    if (fabs(d2) < least) d2 = d2 < 0.0 ? -least : least;
    const double rdv = Rv[3 * kVSquare + j], rd2 = act ? 1.0 / d2 : 0.0;   // a zero column: inf, the class does not settle
    // multipliers, zero on idle lanes
    double fb[MT], f2[MT], gb[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        fb[i] = -b1c[i];
        f2[i] = i < j ? -r2c[i] * rd2 : 0.0;
        if (j < MT) Tc[i * LDT + j] = fb[i];
    }
    __builtin_amdgcn_wave_barrier();
    const double *row = Tc + (j < MT ? j : MT - 1) * LDT;  // the last row of a strict upper triangle is zero
#pragma unroll
    for (int k = 0; k < MT; ++k) gb[k] = act ? row[k] : 0.0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const double scaled = -row_bcast_dyn(rd2, i) * r2c[i];
        if (j < MT) Tc[i * LDT + j] = i < j ? scaled : 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    const auto fv_at = [Rv, j](int i) { return Rv[kVSquare + i * kProjMaxM + j]; };
    const auto gv_at = [Rv, j](int k) { return Rv[2 * kVSquare + k * kProjMaxM + j]; };
    const auto g2_at = [row](int k) { return row[k]; };
    const auto fb_at = [&fb](int i) { return fb[i]; };
    const auto f2_at = [&f2](int i) { return f2[i]; };
    const auto gb_at = [&gb](int k) { return gb[k]; };

    double p = act ? 1.0 + 0.25 * (j % 3) : 0.0;
    double q = act ? 1.0 + 0.25 * ((M + j) % 3) : 0.0;
    double dd_prev = __builtin_inf();
    int since_jump = 0;
    bool settled = false;
    for (int round = 0; round < kRegisterRounds; ++round) {
        double w1 = p * rdv, t = q;                       // forward: w1 = R_V^-T p, t = q - B1^T w1, then w2 = R2^-T t
        TriangularSweeps<0, MT>::forward2(w1, fv_at, t, fb_at);
        double w2 = t * rd2;
        TriangularSweeps<0, MT>::forward(w2, f2_at);
        double qn_raw = w2 * rd2, u = w1;                 // backward: q' = R2^-1 w2, u = w1 - B1 q', then p' = R_V^-1 u
        TriangularSweeps<MT - 1, MT>::backward2(qn_raw, g2_at, u, gb_at);
        double pn_raw = u * rdv;
        TriangularSweeps<MT - 1, MT>::backward(pn_raw, gv_at);
        const double nn = row16_sum(act ? fma(pn_raw, pn_raw, qn_raw * qn_raw) : 0.0);
        const double inv = rcp_normal(sqrt_normal(nn));       // nn = 0, inf or NaN: NaN, the class does not settle
        const double pn = act ? pn_raw * inv : 0.0, qn = act ? qn_raw * inv : 0.0;
        const double dp = pn - p, dq = qn - q;                // z' . z > 0 always: no sign to align
        const double dd = row16_sum(fma(dp, dp, dq * dq));
        const double dd_before = dd_prev;
        settled = settled || dd <= 1e-22 || (dd_prev <= 1e-16 && dd >= 0.25 * dd_prev);
        p = pn;
        q = qn;
        dd_prev = dd;
        ++since_jump;
        if (!settled && since_jump >= 3 && dd < 1e-4 && dd_before < __builtin_inf()) {
            const double r = sqrt(dd / dd_before);
            if (r > 0.05 && r < 0.97) {
                p = fma(r / (1.0 - r), dp, pn);
                q = fma(r / (1.0 - r), dq, qn);
                since_jump = 0;
                dd_prev = __builtin_inf();
            }
        }
        if (__all((settled || !live) ? 1 : 0)) break;     // rows without a class (all zeros) never settle: not waited for
    }
    qv = q;
    return settled;
}

// Algorithm 1 (the homogeneous fit, Q_0 free) for four classes at a time, by one wave, on the factorisations
// V = Q [R_V; 0] of their groups; arguments as for locate_classes_proj, U followed by Q1 and R_V (see kVDoubles).  With H_c = [V | diag(y_c) V] (the sign of the second block
// only flips the sign of Q),
//     Q^T H_c = [ R_V   Q1^T diag(y_c) V ]      Q1^T = rows 0..M-1 of Q^T,
//               [  0     U  diag(y_c) V ]      U    = rows M..n-1,
// so the 2M x 2M triangular factor of H_c is [[R_V, B1], [0, R2]] with B1 = Q1^T diag(y_c) V (M x M) and
// R2 the triangular factor of B2 = U diag(y_c) V ((n-M) x M; n - M >= M by eq. (3)).  B1 and B2 are
// formed as the projected system of Algorithm 2 is (Q1 sits in the 16 rows that follow U in LDS), R2 by the same
// elimination, run over all M columns.  The smallest right singular vector of the assembled factor is found in registers (singular_vector_rows); a class that does not settle there is assembled
// in this wave's scratch, mat[2M][2M+1] | coef[M] | key[n], and goes through the LDS form (homogeneous_q), as many
// classes at a time as the scratch holds (one, as the host sizes it); slot_of(s) tells about class slot s there.
struct ClassSlot {
    int n;                     // available workers, avail[0..n) ascending
    const int *avail;
    int *votes;
};
template <int NB, int RM, int MT, class SlotOf>
__device__ __forceinline__ void locate_classes_hom_proj(const float *y, const float *zeros, const double *U, bool class_live,
                                                        unsigned long long rows, const int *worker_of_row, const double *Pw,
                                                        int M, int A, int *votes, double *scratch, int scratch_doubles,
                                                        SlotOf slot_of) {
    const int lane = lane_id();
    const int j = lane % kClsLanes;
    const double *Rv = U + (ush_rows(RM) + kProjMaxM) * lds_stride(NB);
    double a[RM], b1[MT];
#pragma unroll
    for (int i = 0; i < RM; ++i) a[i] = 0.0;
#pragma unroll
    for (int i = 0; i < MT; ++i) b1[i] = 0.0;
    const float *yj = j < M ? y : zeros;                  // column of this lane: y x^j; idle lanes hold zeros
    const double *wj = Pw + (j < M ? j : 0) * lds_stride(NB);
    project_column<NB>(a, U + (j < RM ? j : 0) * lds_stride(NB), yj, wj);
    project_column<NB>(b1, U + (ush_rows(RM) + j) * lds_stride(NB), yj, wj);
    // R2: the triangular factor of B2 (M <= RM: eq. (3) gives n - M >= M)
    double r2c[MT];
    ClassTriangle<0, MT, RM>::run(a, r2c, M);

    // ---- the singular vector: in registers; classes that do not settle there go through the LDS form below ---------
    const int cl16 = lane / kClsLanes;                    // class slot of this lane in the register layout
    double qv;
    const bool settled = singular_vector_rows<MT>(r2c, b1, Rv, scratch, M, j, cl16, class_live, qv);
    // a_r = Q(x_r) = sum_k q_k x_r^k, rows j, j+16, .. of this lane; the A smallest |a_r| vote
    {
        double qk[MT];
#pragma unroll
        for (int k = 0; k < MT; ++k) qk[k] = row_bcast_dyn(qv, k);              // zero from idle lanes
        constexpr int PR = (NB + kClsLanes - 1) / kClsLanes;
        double key[PR];
#pragma unroll
        for (int pr = 0; pr < PR; ++pr) {
            const int r = j + pr * kClsLanes;
            const double x = Pw[lds_stride(NB) + (r < NB ? r : 0)];
            double av = 0.0;
#pragma unroll
            for (int k = MT - 1; k >= 0; --k) av = fma(av, x, qk[k]);
            key[pr] = ((rows >> r) & 1ull) ? (av == av ? fabs(av) : __builtin_inf()) : __builtin_nan("");
        }
        vote_smallest<PR>(key, A, class_live && settled, worker_of_row, votes);
    }
    const unsigned long long open_lanes = __ballot(class_live && !settled);
    if (open_lanes == 0ull) return;

    // ---- fallback: assemble the factor in LDS and find the vector there (inverse iteration again, then Jacobi) -----
    const int W2 = 2 * M;
    const int LD = W2 + 1;
    const int per_class = W2 * LD + M + NB;
    const int fit = scratch_doubles / per_class;          // >= 1 (hom_scratch_doubles)
    const int cpw = kWave / W2 < fit ? kWave / W2 : fit;  // classes per pass: what the lanes and the scratch hold
    const int clw = lane / W2, jw = lane - clw * W2;      // the layout of homogeneous_q (lane jw owns row jw)
    __builtin_amdgcn_wave_barrier();                      // the transposition scratch is free again
    for (int p0 = 0; p0 < kClsPerWave; p0 += cpw) {
        if (cl16 >= p0 && cl16 < p0 + cpw && j < M) {
            double *mat = scratch + (cl16 - p0) * per_class;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (i < M) {
                    mat[i * LD + j] = Rv[i * kProjMaxM + j];                    // R_V (zero below its diagonal)
                    mat[(M + i) * LD + j] = 0.0;
                    mat[i * LD + M + j] = b1[i];                                // B1
                    mat[(M + i) * LD + M + j] = (i <= j) ? r2c[i] : 0.0;        // R2
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        const bool in_pass = clw < cpw && p0 + clw < kClsPerWave;
        const bool live = in_pass && ((open_lanes >> ((p0 + (in_pass ? clw : 0)) * kClsLanes)) & 1ull) != 0ull;
        double *mat = scratch + (live ? clw : 0) * per_class;
        double *coef = mat + W2 * LD;
        double *key = coef + M;
        homogeneous_q(mat, LD, coef, key, W2, M, jw, live, true);
        const ClassSlot slot = slot_of(p0 + (live ? clw : 0));
        if (live) {
            for (int r = jw; r < slot.n; r += W2) {       // a_r = Q(x_r), Q_k = coef[k]
                const double x = Pw[lds_stride(NB) + (worker_of_row != nullptr ? r : slot.avail[r])];
                double av = 0.0;
                for (int t = M - 1; t >= 0; --t) av = fma(av, x, coef[t]);
                key[r] = (av != av) ? __builtin_inf() : fabs(av);
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (live) pick_and_vote(key, slot.avail, slot.n, A, jw, W2, slot.votes);
        __builtin_amdgcn_wave_barrier();
    }
}

// Per-wave LDS scratch of Algorithm 1's locator: the transposition tiles of singular_vector_rows (4 classes x MT x
// (MT + 1)) or, for a class that falls back to homogeneous_q, ONE assembled factor with its coefficient and key
// arrays.  Kept this small on purpose: LDS, not registers, decides how many groups a CU holds (at K = 8, A = 2 with
// three factors per wave seven workgroups fitted a CU where eight were due, and the launch took two rounds).
__host__ __device__ constexpr int hom_scratch_doubles(int M, int rows, int MT) {
    const int fallback = 2 * M * (2 * M + 1) + M + rows;
    const int transpose = kClsPerWave * MT * (MT + 1);
    const int most = fallback > transpose ? fallback : transpose;
    return (most + 1) & ~1;
}

// Doubles of the shared factorisation as the kernel keeps it in LDS (and as full_basis_kernel writes it out):
// Ush[ush_rows(RM)][lds_stride(NB)], and for Algorithm 1's locator also Q1sh[16][lds_stride(NB)] | Rv[16][16].
template <int NB, int RM, bool HOMOG>
constexpr int basis_doubles() {
    return (ush_rows(RM) + (HOMOG ? kProjMaxM : 0)) * lds_stride(NB) + (HOMOG ? kProjMaxM * kProjMaxM : 0);
}
// The same between LDS and the caller's workspace, where rows have stride basis_stride(NB).
template <int NB, int RM, bool HOMOG>
__device__ __forceinline__ void basis_from_workspace(double *Ush, const double *__restrict__ basis) {
    constexpr int rows = ush_rows(RM) + (HOMOG ? kProjMaxM : 0);
    for (int e = threadIdx.x; e < rows * NB; e += blockDim.x)
        Ush[e / NB * lds_stride(NB) + e % NB] = basis[e / NB * basis_stride(NB) + e % NB];
    if (HOMOG)
        for (int e = threadIdx.x; e < kProjMaxM * kProjMaxM; e += blockDim.x)
            Ush[rows * lds_stride(NB) + e] = basis[rows * basis_stride(NB) + e];
}
template <int NB, int RM, bool HOMOG>
__device__ __forceinline__ void basis_to_workspace(const double *Ush, double *__restrict__ basis) {
    constexpr int rows = ush_rows(RM) + (HOMOG ? kProjMaxM : 0);
    for (int e = threadIdx.x; e < rows * NB; e += blockDim.x)
        basis[e / NB * basis_stride(NB) + e % NB] = Ush[e / NB * lds_stride(NB) + e % NB];
    if (HOMOG)
        for (int e = threadIdx.x; e < kProjMaxM * kProjMaxM; e += blockDim.x)
            basis[rows * basis_stride(NB) + e] = Ush[rows * lds_stride(NB) + e];
}

// HOMOG: Algorithm 1's fit as the per-class locator (locate_classes_hom_proj) instead of Algorithm 2's.
// dynamic LDS (doubles): basis (see basis_doubles; HOMOG: up to kVDoubles) | Pw[16][lds_stride] | xs[NB] | float Ysh[CW + 1][y_stride]
//               | WdT[(n_cap-A)*KP] | alpha_s[K] | beta_s[N] | HOMOG: scratch[nw][hom_scratch_doubles]
//               then ints: avail[N] | F[N] | Fpos[N] | votes[N] | n | flag
template <int NB, int RM, bool HOMOG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(!HOMOG && RM <= 16 && NB <= 28 ? 3 : 2))) void decode_byzantine_proj_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out,
    int32_t *__restrict__ adv, int32_t *__restrict__ status, int K, int N, int S, int A, int64_t C, int64_t Cv,
    int vec4, int sign_mode, int n_cap, int cw_log2, int splits, int32_t *__restrict__ workspace,
    const double *__restrict__ full_basis, const Nodes nodes) {
    extern __shared__ __align__(16) double lds_d[];
    const int KP = round_up4(K);
    const int M = K + A;
    const int nw = blockDim.x / kWave;
    const int CW = 1 << cw_log2;                          // classes per staged tile (16, 32 or 64)
    double *Ush = lds_d;
    constexpr int kUshDoubles = basis_doubles<NB, RM, HOMOG>();
    constexpr int YS = y_stride(NB);
    double *Q1sh = Ush + ush_rows(RM) * lds_stride(NB);   // HOMOG only: the 16 rows after U, then R_V
    double *Rv = Q1sh + kProjMaxM * lds_stride(NB);
    double *Pw = Ush + kUshDoubles + (HOMOG ? kVDoubles - kVSquare : 0);
    double *xs = Pw + kPowers * lds_stride(NB);
    float *Ysh = reinterpret_cast<float *>(xs + NB);      // [CW + 1][YS], the last row stays zero
    double *WdT = xs + NB + (CW + 1) * YS / 2;
    double *alpha_s = WdT + (n_cap - A) * KP;
    double *beta_s = alpha_s + K;
    const int hom_wave_doubles = HOMOG ? hom_scratch_doubles(M, NB, hom_mt(NB)) : 0;
    double *hom_scratch = beta_s + N;
    int *avail = reinterpret_cast<int *>(hom_scratch + static_cast<size_t>(nw) * hom_wave_doubles);
    int *F = avail + N;
    int *Fpos = F + N;
    int *votes = Fpos + N;
    int *n_sh = votes + N;

    // splits > 1: `splits` workgroups share a group, workgroup `part` taking the class tiles part, part + splits, ..
    const int64_t g = blockIdx.x / splits;
    const int part = static_cast<int>(blockIdx.x - g * splits);
    const int wv = wave_id();
    const int tid = threadIdx.x;
    const float *pg = preds + static_cast<size_t>(g) * N * C;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = tid; e < (n_cap - A) * KP; e += blockDim.x) WdT[e] = 0.0;
    for (int e = tid; e < N; e += blockDim.x) votes[e] = 0;
    if (wv == 0) {
        const int cnt = survivors_from_mask(mask + g * N, N, avail);
        if (lane_id() == 0) *n_sh = cnt;
    }
    __syncthreads();
    const int n = *n_sh;
    const bool good = S < 0 ? (n >= 2 * M && n <= n_cap) : n == n_cap;
    if (tid == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;
    // A group in which every worker answered has the node set of the whole call: its complement basis was
    // factorised once, ahead of this launch (full_basis_kernel), and is only copied here.
    const bool preloaded = full_basis != nullptr && n == N;
    if (preloaded) basis_from_workspace<NB, RM, HOMOG>(Ush, full_basis);
    else
        for (int e = tid; e < kUshDoubles; e += blockDim.x) Ush[e] = 0.0;
    for (int e = tid; e < YS; e += blockDim.x) Ysh[CW * YS + e] = 0.0f;

    // first class tile: the loads are issued now and land in LDS after the shared factorisation
    constexpr int kPrefetch = 8;
    const int64_t cb_first = static_cast<int64_t>(part) * CW;
    const int slots = NB * CW;                            // slot = (row r, class c) = (slot >> cw_log2, slot & (CW-1))
    float pf[kPrefetch];
#pragma unroll
    for (int u = 0; u < kPrefetch; ++u) {
        const int slot = tid + u * blockDim.x;
        const int r = slot >> cw_log2, c = slot & (CW - 1);
        pf[u] = (slot < slots && r < n && cb_first + c < C) ? pg[static_cast<size_t>(avail[r]) * C + cb_first + c] : 0.0f;
    }

    // powers of the available workers' nodes, x^e by repeated multiplication; rows past n are zero
    for (int r = tid; r < NB; r += blockDim.x) {
        const double x = r < n ? beta_s[avail[r]] : 0.0;
        if (r < n) xs[r] = x;
        double p = r < n ? 1.0 : 0.0;
        for (int e = 0; e < kPowers; ++e) {
            Pw[e * lds_stride(NB) + r] = p;
            p *= x;
        }
    }
    __syncthreads();
    if (wv == 0 && !preloaded) shared_complement_basis<NB, RM, HOMOG>(Pw, n, M, Ush, Q1sh, Rv);
    if (HOMOG) {
        __syncthreads();
        for (int e = tid; e < kVSquare; e += blockDim.x) sweep_multipliers(Rv, e, M);
    }

    for (int64_t cb = cb_first; cb < C; cb += static_cast<int64_t>(splits) * CW) {   // class tiles of this part
        if (cb == cb_first) {
#pragma unroll
            for (int u = 0; u < kPrefetch; ++u) {
                const int slot = tid + u * blockDim.x;
                if (slot < slots) Ysh[(slot & (CW - 1)) * YS + (slot >> cw_log2)] = pf[u];
            }
            for (int slot = tid + kPrefetch * blockDim.x; slot < slots; slot += blockDim.x) {
                const int r = slot >> cw_log2, c = slot & (CW - 1);
                Ysh[c * YS + r] = (r < n && cb + c < C) ? pg[static_cast<size_t>(avail[r]) * C + cb + c] : 0.0f;
            }
        } else {
            __syncthreads();                              // every wave is done with the previous tile
            for (int slot = tid; slot < slots; slot += blockDim.x) {
                const int r = slot >> cw_log2, c = slot & (CW - 1);
                Ysh[c * YS + r] = (r < n && cb + c < C) ? pg[static_cast<size_t>(avail[r]) * C + cb + c] : 0.0f;
            }
        }
        __syncthreads();
        const int tile_classes = (C - cb < CW) ? static_cast<int>(C - cb) : CW;
        for (int c_rel = wv * kClsPerWave; c_rel < tile_classes; c_rel += nw * kClsPerWave) {
            if (HOMOG)
                locate_classes_hom_proj<NB, RM, hom_mt(NB)>(Ysh + (c_rel + lane_id() / kClsLanes) * YS, Ysh + CW * YS, Ush,
                                                c_rel + lane_id() / kClsLanes < tile_classes, (1ull << n) - 1ull, avail, Pw, M, A,
                                                votes, hom_scratch + static_cast<size_t>(wv) * hom_wave_doubles,
                                                hom_wave_doubles, [=](int) { return ClassSlot{n, avail, votes}; });
            else
                locate_classes_proj<NB, RM>(Ysh + (c_rel + lane_id() / kClsLanes) * YS, Ysh + CW * YS, Ush,
                                            c_rel + lane_id() / kClsLanes < tile_classes, (1ull << n) - 1ull, avail, Pw, M, A,
                                            votes);
        }
    }
    __syncthreads();

    float *og = out + static_cast<size_t>(g) * K * C;
    if (splits > 1 && !pool_votes_last_arrival(workspace + g * (N + 1), votes, N, splits, n_sh + 1)) return;
    const bool staged = C <= CW;                          // the one tile holds every prediction of the group
    select_adversaries(adv + g * A, avail, n, N, A, votes, F, Fpos);
    const int nF = n - A;
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();
    if (staged) {
        // out[j][c] = sum_r WdT[r][j] * Y[F_r][c] straight from the staged tile
        const int Ci = static_cast<int>(C);
        for (int o = tid; o < K * Ci; o += blockDim.x) {
            const int jq = o / Ci, c = o - jq * Ci;
            double acc = 0.0;
#pragma unroll 6
            for (int r = 0; r < nF; ++r)
                acc = fma(WdT[r * KP + jq], static_cast<double>(Ysh[c * YS + Fpos[r]]), acc);
            og[o] = static_cast<float>(acc);
        }
    } else if (vec4) {
        contract_group<4>(pg, og, F, nF, K, KP, C, Cv, WdT);
    } else {
        contract_group<1>(pg, og, F, nF, K, KP, C, Cv, WdT);
    }
}

// Algorithm 2 for groups of at most fifteen classes (the paper's Byzantine operating points, Section 4.2, have ten).
// A workgroup of up to four waves takes GPW = 1, 2 or 4 consecutive groups and walks their GPW * C classes four at a time, so
// that class slots are filled across groups (ten classes: four groups fill ten rounds where each alone needs three,
// twelve slots for ten classes).  Rows are workers, not survivors: the predictions are staged as they lie, with zeros
// for missing answers, all groups use one table of powers, and a missing worker is a zero column of its group's U.
// U comes from the call's one factorisation (SHARED: no stragglers, see full_basis_kernel; without a workspace the first
// wave forms the same one, bit for bit) or from the first wave, which factorises the workgroup's groups side by side, a
// 16-lane row each.
// The decode at the end is one product on the float64 matrix cores per group: with T[j][i] = 1 / (alpha_j - beta_i),
// which depends on the nodes only, and s_i = the alternating sign of worker i, 0 if it does not count,
//     out[j][c] = (sum_i T[j][i] s_i y_ic) / (sum_i T[j][i] s_i):
// column 15 of the product carries the denominators (C <= 15).  A query node that is a worker's node has T = 0 there and
// takes that worker's row as it is, if the worker counts.
// K = 8, A = 2, 20 of 24 workers, 2048 groups of 10 classes: 24.5 us with a workgroup per group, 19.9 us this way;
// K = 12, A = 2, 28 workers, 8192 groups: 91.2 us with this packing but decoder weights per group, 68.3 us.
// NB >= N - S bounds the workers that answer, NW >= N all workers, RM >= N - S - M.
// HOMOG: Algorithm 1's locator instead (locate_classes_hom_proj): K = 8, 2048 groups 61 us with a workgroup per group
// and the sweeps' broadcasts as moves, 47.5 us; K = 12, 8192 groups 357 and 183 us.
// dynamic LDS: double basis[SHARED ? 1 : GPW][packed_basis_doubles] | Pw[16][lds_stride(NW)] | T[16][NW + 1] | sgn[GPW][NW]
//              | HOMOG: scratch[nw][hom_scratch_doubles]
//              | float Ysh[16 GPW + 1][y_stride(NW)] (the last row stays zero: empty class slots read it)
//              | uint64 bits[GPW] | int avail[GPW][NW] | votes[GPW][64] | hit[16]
template <int NB, int RM, int NW, bool HOMOG>
constexpr int packed_basis_doubles() {                   // U, and for Algorithm 1 Q1 and what kVDoubles lists
    return basis_doubles<NW, RM, HOMOG>() + (HOMOG ? kVDoubles - kVSquare : 0);
}
template <int NB, int RM, int NW, bool HOMOG>
constexpr size_t packed_lds_bytes(bool shared, int gpw, int nw, int M) {
    return sizeof(double) * (static_cast<size_t>(shared ? 1 : gpw) * packed_basis_doubles<NB, RM, NW, HOMOG>() +
                             kPowers * lds_stride(NW) + 16 * (NW + 1) + gpw * NW + gpw +
                             (HOMOG ? nw * hom_scratch_doubles(M, NW, hom_mt(NB)) : 0)) +
           sizeof(float) * (static_cast<size_t>(gpw * kClsLanes + 1) * y_stride(NW)) +
           sizeof(int) * (static_cast<size_t>(gpw) * (NW + kWave) + 16);
}
constexpr int kPackedWaves = 4;      // at most

template <int NB, int RM, int NW, bool SHARED, bool HOMOG>
__global__ __launch_bounds__(kPackedWaves * kWave) __attribute__((amdgpu_waves_per_eu(!HOMOG && NB <= 28 ? 3 : 2))) void decode_byzantine_packed_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out,
    int32_t *__restrict__ adv, int32_t *__restrict__ status, int64_t G, int K, int N, int S, int n_cap, int A, int C,
    int sign_mode, int gpw, const double *__restrict__ full_basis, const Nodes nodes) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) double lds_d[];
    constexpr int CW = kClsLanes;
    constexpr int YS = y_stride(NW);
    constexpr int kStride = lds_stride(NW);
    constexpr int kQ1 = ush_rows(RM) * kStride;           // inside a basis: U, then Q1, then R_V
    constexpr int kRv = kQ1 + kProjMaxM * kStride;
    constexpr int kBasis = packed_basis_doubles<NB, RM, NW, HOMOG>();
    constexpr int TS = NW + 1;                            // odd: the sixteen rows an operand load touches lie in distinct banks
    const int threads = blockDim.x;                       // at least a wave per group
    const int nw = threads / kWave;
    const int M = K + A;
    double *Ush = lds_d;
    double *Pw = Ush + (SHARED ? 1 : gpw) * kBasis;
    double *T = Pw + kPowers * kStride;
    double *sgn = T + 16 * TS;
    const int hom_doubles = HOMOG ? hom_scratch_doubles(M, NW, hom_mt(NB)) : 0;
    double *hom_scratch = sgn + gpw * NW;
    float *Ysh = reinterpret_cast<float *>(hom_scratch + nw * hom_doubles);
    float *zeros = Ysh + gpw * CW * YS;
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(zeros + YS);
    int *avail = reinterpret_cast<int *>(bits + gpw);
    int *votes = avail + gpw * NW;
    int *hit = votes + gpw * kWave;
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * gpw;
    const int here = G - g0 < gpw ? static_cast<int>(G - g0) : gpw;   // groups of this workgroup
    const int tid = threadIdx.x;
    const int wv = wave_id();
    const int lane = lane_id();
    const int c_ld = tid & (CW - 1);

    if (wv < gpw) {                                       // N <= 48: one ballot reads a mask row
        const int q = wv;
        const bool b = q < here && lane < N && mask[(g0 + q) * N + lane] != 0;
        unsigned long long m = __ballot(b);
        const int n = static_cast<int>(__popcll(m));
        const bool good = q < here && (S < 0 ? (n >= 2 * M && n <= n_cap) : n == n_cap);
        if (lane == 0 && q < here && status != nullptr) status[g0 + q] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
        if (!good) m = 0ull;
        if (lane == 0) bits[q] = m;
        if (b && good) avail[q * NW + __popcll(m & ((1ull << lane) - 1ull))] = lane;
        votes[q * kWave + lane] = 0;
    }
    if (SHARED && full_basis != nullptr) {
        basis_from_workspace<NB, RM, HOMOG>(Ush, full_basis);
    } else {
        for (int e = tid; e < (SHARED ? 1 : gpw) * kBasis; e += threads) Ush[e] = 0.0;
    }
    if (tid < NW) {
        const double x = tid < N ? nodes.beta[tid] : 0.0;
        double pw = tid < N ? 1.0 : 0.0;
        for (int e = 0; e < kPowers; ++e) {
            Pw[e * kStride + tid] = pw;
            pw *= x;
        }
    }
    if (tid >= threads - 16) hit[tid - (threads - 16)] = -1;
    __syncthreads();
    // predictions: row slot u of this thread is row tid / 16 + u * (threads / 16) of the stacked [gpw][NW] tiles;
    // a pass takes four rows per wave and there are gpw waves or more, so NW / 4 passes do.  Only rows of workers that
    // answered are read; T is evaluated while they are on their way.  (Kept in registers until the first wave has
    // factorised they cost it 16 to 45 registers; a mask byte per lane and row, to load ahead of the barrier: 20.4 us at
    // K = 8, 2048 groups, and 69.6 at K = 12, 8192 groups, against 19.9 and 68.2 this way.)
    const int rows_per_pass = threads / CW;
    float pf[NW / 4];
#pragma unroll
    for (int u = 0; u < NW / 4; ++u) {
        const int R = tid / CW + u * rows_per_pass;
        const int q = R / NW, r = R % NW;
        const bool there = q < gpw && ((bits[q] >> r) & 1ull) != 0ull;
        pf[u] = (there && c_ld < C) ? preds[(static_cast<size_t>(g0 + q) * N + r) * C + c_ld] : 0.0f;
    }
    for (int e = tid; e < 16 * NW; e += threads) {
        const int j = e / NW, i = e - j * NW;
        const bool in = j < K && i < N;
        const double d = in ? nodes.alpha[in ? j : 0] - nodes.beta[in ? i : 0] : 1.0;
        if (d == 0.0) hit[j] = i;                         // nodes are distinct: at most one
        T[j * TS + i] = (in && d != 0.0) ? 1.0 / d : 0.0;
    }
#pragma unroll
    for (int u = 0; u < NW / 4; ++u) {
        const int R = tid / CW + u * rows_per_pass;
        const int q = R / NW, r = R % NW;
        if (q < gpw) Ysh[(q * CW + c_ld) * YS + r] = pf[u];
    }
    for (int e = tid; e < YS; e += threads) zeros[e] = 0.0f;
    if (SHARED && full_basis == nullptr && wv == 0) {
        if constexpr (NB == NW) shared_complement_basis<NB, RM, HOMOG>(Pw, N, M, Ush, Ush + kQ1, Ush + kRv);
    }
    if (!SHARED && wv == 0) {
        const int q = lane / kClsLanes < gpw ? lane / kClsLanes : 0;
        const int n = lane / kClsLanes < gpw ? static_cast<int>(__popcll(bits[q])) : 0;
        double *basis = Ush + q * kBasis;
        rows_complement_basis<NB, HOMOG>(Pw, avail + q * NW, n, M, basis, kStride, basis + kQ1, basis + kRv);
    }
    __syncthreads();
    if (HOMOG) {
        for (int e = tid; e < (SHARED ? 1 : here) * kVSquare; e += threads)
            sweep_multipliers(Ush + e / kVSquare * kBasis + kRv, e % kVSquare, M);
        __syncthreads();
    }

    const int total = gpw * C;
    for (int c0 = wv * kClsPerWave; c0 < total; c0 += nw * kClsPerWave) {
        const int slot = c0 + lane / kClsLanes;           // the class of this lane's row
        const int q = slot < total ? slot / C : 0;
        const unsigned long long rows = bits[q];
        const bool live = slot < total && rows != 0ull;
        const float *y = live ? Ysh + (q * CW + slot - q * C) * YS : zeros;
        const double *basis = SHARED ? Ush : Ush + q * kBasis;
        if constexpr (HOMOG)
            locate_classes_hom_proj<NW, RM, hom_mt(NB)>(
                y, zeros, basis, live, rows, nullptr, Pw, M, A, votes + q * kWave, hom_scratch + wv * hom_doubles, hom_doubles,
                [=](int s) {
                    const int qs = c0 + s < total ? (c0 + s) / C : 0;
                    return ClassSlot{static_cast<int>(__popcll(bits[qs])), avail + qs * NW, votes + qs * kWave};
                });
        else
            locate_classes_proj<NW, RM>(y, zeros, basis, live, rows, nullptr, Pw, M, A, votes + q * kWave);
    }
    __syncthreads();

    if (wv >= here || bits[wv] == 0ull) return;           // a wave per group from here on, no barrier left
    {
        const int q = wv;
        const unsigned long long below = (1ull << lane) - 1ull;
        // the A most voted workers, equal counts: smaller index first.  Every class gives A distinct workers a vote, so
        // at least A have one.
        int key = lane < N ? (votes[q * kWave + lane] << 6) | (kWave - 1 - lane) : -1;
        unsigned long long drop = 0ull;
        for (int pick = 0; pick < A; ++pick) {
            int m = key;
            m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor1, 0xF, 0xF, true));
            m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor2, 0xF, 0xF, true));
            m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowHalfMirror, 0xF, 0xF, true));
            m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowMirror, 0xF, 0xF, true));
            m = max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
                    max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
            const int w = kWave - 1 - (m & (kWave - 1));
            drop |= 1ull << w;
            if (lane == w) key = -1;
        }
        if ((drop >> lane) & 1ull) adv[(g0 + q) * A + __popcll(drop & below)] = lane;
        const unsigned long long left = bits[q] & ~drop;
        if (lane < NW) {
            const int odd = sign_mode == APPROXIFER_SIGN_SURVIVOR_RANK ? static_cast<int>(__popcll(left & below)) & 1 : lane & 1;
            sgn[q * NW + lane] = ((left >> lane) & 1ull) ? (odd ? -1.0 : 1.0) : 0.0;
        }
        __builtin_amdgcn_wave_barrier();
        const int c = lane & 15, k = lane >> 4;
        const float *y = Ysh + (q * CW + c) * YS;         // this lane's class column
        v4d acc[2] = {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int s = 0; s < NW / 4; ++s) {
            const int i = 4 * s + k;
            const double sg = sgn[q * NW + i];
            const double v = c == 15 ? 1.0 : static_cast<double>(y[i]);
            acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(T[c * TS + i], sg != 0.0 ? sg * v : 0.0, acc[s & 1], 0, 0, 0);
        }
        float *og = out + static_cast<size_t>(g0 + q) * K * C;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int j = 4 * t + k;
            const double num = acc[0][t] + acc[1][t];
            const double den = row_bcast<15>(num);
            double v = num / den;
            const int h = hit[j];
            if (h >= 0 && ((left >> h) & 1ull) != 0ull) v = static_cast<double>(y[h]);
            if (j < K && c < C) og[j * C + c] = static_cast<float>(v);
        }
    }
}

// The complement basis of the node set of ALL N workers, once per call, for the groups whose mask is full (the
// paper's Byzantine experiments have no stragglers: every group then shares this one factorisation).  One wave;
// writes it to `basis`, rows of stride basis_stride(NB).
template <int NB, int RM, bool HOMOG>
__global__ __launch_bounds__(kWave) void full_basis_kernel(double *__restrict__ basis, int N, int M, const Nodes nodes) {
    constexpr int kUshDoubles = basis_doubles<NB, RM, HOMOG>();
    __shared__ double Ush[kUshDoubles];
    __shared__ double Pw[kPowers * lds_stride(NB)];
    const int tid = threadIdx.x;
    for (int e = tid; e < kUshDoubles; e += kWave) Ush[e] = 0.0;
    for (int r = tid; r < NB; r += kWave) {
        const double x = r < N ? nodes.beta[r] : 0.0;
        double p = r < N ? 1.0 : 0.0;
        for (int e = 0; e < kPowers; ++e) {
            Pw[e * lds_stride(NB) + r] = p;
            p *= x;
        }
    }
    __syncthreads();
    shared_complement_basis<NB, RM, HOMOG>(Pw, N, M, Ush, Ush + ush_rows(RM) * lds_stride(NB),
                                           Ush + (ush_rows(RM) + kProjMaxM) * lds_stride(NB));
    __syncthreads();
    basis_to_workspace<NB, RM, HOMOG>(Ush, basis);
}

// ------------------------------------------------------------------------------------------------
// general kernel: the full system per class, in LDS
// ------------------------------------------------------------------------------------------------
// Appendix A, Algorithm 3, for the classes c0 .. c0+cpw-1 of one group, by one wave: the same least-squares fit of
// (P, Q) as Algorithm 2, then the K values r(alpha_j) = P(alpha_j) / Q(alpha_j) instead of an error locator.
// Layout as locate_classes_wave (per class  mat[n][2M] | sol[2M-1] in the coef and key slots); lane j of a class
// evaluates query j, so K <= 2M lanes always suffice.
__device__ __forceinline__ void reconstruct_classes_wave(const float *__restrict__ pg, float *__restrict__ og, int64_t C,
                                                         int64_t c0, int cpw, const int *avail, const double *xs,
                                                         const double *alpha_s, int n, int K, int M, double *scratch) {
    const int lane = lane_id();
    const int W2 = 2 * M;
    const int cols = W2 - 1;                 // unknowns P_0..P_{M-1}, Q_1..Q_{M-1}; column `cols` is the rhs
    const int cl = lane / W2;
    const int j = lane - cl * W2;
    const int64_t c = c0 + cl;
    const bool live = cl < cpw && c < C;
    const int per_class = n * W2 + M + n;    // M + n >= 3M > cols doubles follow the matrix
    double *mat = scratch + (live ? cl : 0) * per_class;
    double *sol = mat + n * W2;

    build_class_system(pg, C, c, avail, xs, n, M, mat, W2, j, W2, live);
    factor_class_system(mat, W2, n, j, cols, live);

    // back substitution for every unknown; lane j holds the transformed right-hand side entry of row j
    double s = (live && j < cols) ? mat[j * W2 + cols] : 0.0;
    const double diag = (live && j < cols) ? mat[j * W2 + j] : 1.0;
    for (int t = cols - 1; t >= 0; --t) {
        if (live && j == t) sol[t] = s / diag;
        __builtin_amdgcn_wave_barrier();
        const double v = sol[t];
        if (live && j < t) s = fma(-mat[j * W2 + t], v, s);
        __builtin_amdgcn_wave_barrier();
    }
    if (live && j < K) {
        const double z = alpha_s[j];
        double num = 0.0, den = 0.0;
        for (int k = M - 1; k >= 0; --k) num = fma(num, z, sol[k]);              // P_0 .. P_{M-1}
        for (int k = M - 1; k >= 1; --k) den = fma(den, z, sol[M - 1 + k]);      // Q_1 .. Q_{M-1}
        den = fma(den, z, 1.0);                                                  // Q_0 = 1
        og[static_cast<size_t>(j) * C + c] = static_cast<float>(num / den);
    }
    __builtin_amdgcn_wave_barrier();
}

// One workgroup per group; waves take the classes cpw at a time.
// dynamic LDS: double scratch[nw][cpw * (n*2M + M + n)] | double xs[n] | double alpha_s[K] | double beta_s[N] | int avail[N] | int n
__global__ void decode_rational_kernel(const float *__restrict__ preds, const uint8_t *__restrict__ mask,
                                       float *__restrict__ out, int32_t *__restrict__ status, int K, int N, int S, int A,
                                       int64_t C, int cpw, int n_cap, const Nodes nodes) {
    extern __shared__ __align__(16) double lds_d[];
    const int M = K + A;
    const int nw = blockDim.x / kWave;
    const int wave_doubles = cpw * (n_cap * 2 * M + M + n_cap);
    double *scratch = lds_d;
    double *xs = scratch + static_cast<size_t>(nw) * wave_doubles;
    double *alpha_s = xs + n_cap;
    double *beta_s = alpha_s + K;
    int *avail = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = avail + N;
    const int64_t g = blockIdx.x;
    const int wv = wave_id();

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    if (wv == 0) {
        const int cnt = survivors_from_mask(mask + g * N, N, avail);
        if (lane_id() == 0) *n_sh = cnt;
    }
    __syncthreads();
    const int n = *n_sh;
    const bool good = S < 0 ? (n >= 2 * M && n <= n_cap) : n == n_cap;
    if (threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;
    for (int r = threadIdx.x; r < n; r += blockDim.x) xs[r] = beta_s[avail[r]];
    __syncthreads();
    const float *pg = preds + static_cast<size_t>(g) * N * C;
    float *og = out + static_cast<size_t>(g) * K * C;
    for (int64_t c0 = static_cast<int64_t>(wv) * cpw; c0 < C; c0 += static_cast<int64_t>(nw) * cpw)
        reconstruct_classes_wave(pg, og, C, c0, cpw, avail, xs, alpha_s, n, K, M, scratch + static_cast<size_t>(wv) * wave_doubles);
}

// dynamic LDS: double scratch[nw][cpw * (n*LD + M + n)] (LD = 2M, 2M+1 for Algorithm 1) | double WdT[(n-A) * KP] | double xs[n]
//              | double alpha_s[K] | double beta_s[N]
//              | int avail[N] | int F[N] | int Fpos[N] | int votes[N] | int n | int flag
template <bool HOMOG>
__global__ void decode_byzantine_general_kernel(const float *__restrict__ preds, const uint8_t *__restrict__ mask,
                                                float *__restrict__ out, int32_t *__restrict__ adv,
                                                int32_t *__restrict__ status, int K, int N, int S, int A, int64_t C,
                                                int64_t Cv, int vec4, int sign_mode, int cpw, int n_cap,
                                                int splits, int32_t *__restrict__ workspace, const Nodes nodes) {
    extern __shared__ __align__(16) double lds_d[];
    const int KP = round_up4(K);
    const int M = K + A;
    const int nF_cap = n_cap - A;
    const int nw = blockDim.x / kWave;
    const int wave_doubles = cpw * (n_cap * (HOMOG ? 2 * M + 1 : 2 * M) + M + n_cap);

    double *scratch = lds_d;
    double *WdT = scratch + static_cast<size_t>(nw) * wave_doubles;
    double *xs = WdT + nF_cap * KP;
    double *alpha_s = xs + n_cap;
    double *beta_s = alpha_s + K;
    int *avail = reinterpret_cast<int *>(beta_s + N);
    int *F = avail + N;
    int *Fpos = F + N;
    int *votes = Fpos + N;
    int *n_sh = votes + N;

    // splits > 1: `splits` workgroups share a group, see pool_votes_last_arrival
    const int64_t g = blockIdx.x / splits;
    const int part = static_cast<int>(blockIdx.x - g * splits);
    const int wv = wave_id();
    const float *pg = preds + static_cast<size_t>(g) * N * C;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < nF_cap * KP; e += blockDim.x) WdT[e] = 0.0;
    for (int e = threadIdx.x; e < N; e += blockDim.x) votes[e] = 0;
    if (wv == 0) {
        const int cnt = survivors_from_mask(mask + g * N, N, avail);
        if (lane_id() == 0) *n_sh = cnt;
    }
    __syncthreads();
    const int n = *n_sh;
    const bool good = S < 0 ? (n >= 2 * M && n <= n_cap) : n == n_cap;
    if (threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    for (int r = threadIdx.x; r < n; r += blockDim.x) xs[r] = beta_s[avail[r]];
    __syncthreads();
    for (int64_t c0 = (static_cast<int64_t>(part) * nw + wv) * cpw; c0 < C; c0 += static_cast<int64_t>(splits) * nw * cpw)
        locate_classes_wave<HOMOG>(pg, C, c0, cpw, avail, xs, n, M, A, scratch + static_cast<size_t>(wv) * wave_doubles,
                                   votes);
    __syncthreads();
    if (splits > 1 && !pool_votes_last_arrival(workspace + g * (N + 1), votes, N, splits, n_sh + 1)) return;

    finish_group(pg, out + static_cast<size_t>(g) * K * C, adv + g * A, avail, n, N, A, K, KP, C, Cv, vec4 != 0, sign_mode,
                 alpha_s, beta_s, votes, F, Fpos, WdT);
}

// Before a launch in which several workgroups share a group: zero the workspace words through which they meet.
// (A kernel, not a memset: the call may be recorded into a HIP graph.)
__global__ void clear_workspace_kernel(int32_t *__restrict__ workspace, int64_t words) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < words) workspace[i] = 0;
}

// Locates the liars of groups by the votes of their classes (`votes`: N counters of N + 1 words a group, from the launch before) and
// decodes: a workgroup to 64 vector columns of a group.  A launch of its own where a group has many classes: one workgroup decoding
// all of a group, K = 8, A = 3, 26 workers, 55 groups of 787 classes took 116 us, 37 this way.
// dynamic LDS: double WdT[nF KP] | alpha_s[K] | beta_s[N] | int F[N]
size_t located_lds_bytes(int K, int N, int nF) {
    return sizeof(double) * (static_cast<size_t>(nF) * ((K + 3) & ~3) + K + N) + sizeof(int) * N;
}
template <int VEC>
__global__ __launch_bounds__(kPairThreads) void decode_located_kernel(const float *__restrict__ preds, const uint8_t *__restrict__ mask,
                                                                      const int32_t *__restrict__ votes, float *__restrict__ out,
                                                                      int32_t *__restrict__ adv, int32_t *__restrict__ status, int K,
                                                                      int N, int S, int A, int64_t C, int64_t Cv, int64_t tiles,
                                                                      int sign_mode, const Nodes nodes) {
    extern __shared__ __align__(16) double lds_d[];
    const int KP = round_up4(K), nF = N - S - A, lane = lane_id();
    double *WdT = lds_d, *alpha_s = WdT + nF * KP, *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    const int64_t g = blockIdx.x / tiles, tile = blockIdx.x - g * tiles;
    const unsigned long long there = __ballot(lane < N && mask[g * N + lane] != 0);       // N < 64
    const unsigned long long drop = most_voted(votes + g * (N + 1), N, A), left = there & ~drop, below = (1ull << lane) - 1ull;
    stage_nodes(nodes, K, N, alpha_s, beta_s);
    const bool good = static_cast<int>(__popcll(there)) == N - S;
    if (tile == 0 && threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;
    if (tile == 0 && wave_id() == 0 && ((drop >> lane) & 1ull)) adv[g * A + __popcll(drop & below)] = lane;
    for (int e = threadIdx.x; e < nF * KP; e += kPairThreads) WdT[e] = 0.0;
    if (wave_id() == 0 && ((left >> lane) & 1ull)) F[__popcll(left & below)] = lane;
    __syncthreads();
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();
    const int64_t cv0 = tile * kColsPerTile;
    typename PredVec<VEC>::type unused[kRowChunk];
    contract_tile<VEC, false>(preds + static_cast<size_t>(g) * N * C, out + static_cast<size_t>(g) * K * C, F, nF, K, KP, C, cv0,
                              cv0 + kColsPerTile < Cv ? cv0 + kColsPerTile : Cv, WdT, unused);
}

// ---- launch shapes (host) --------------------------------------------------------------------------
constexpr int64_t kFillWaves = 4096;     // waves that put about four on every SIMD of the chip (256 CUs x 4 SIMDs)

bool proj_domain(int M, int n) { return M <= kProjMaxM && n <= 48 && n - M <= 32; }

struct ProjShape {
    int cw_log2, nw, splits;
};
// `may_split`: the caller brought a workspace for the workgroups of a group to meet in.
ProjShape proj_shape(int64_t G, int64_t C, bool may_split, int64_t fill_waves = kFillWaves) {
    ProjShape p;
    p.cw_log2 = C <= 16 ? 4 : (C <= 32 ? 5 : 6);           // classes per staged tile: 16, 32 or 64
    const int CW = 1 << p.cw_log2;
    // waves per workgroup: one per four classes of a tile, at most four -- but no more than it takes to put
    // about four waves on every SIMD of the chip: beyond that, extra waves of a group only
    // idle through the shared factorisation (measured at G = 2048, C = 10: 1 wave 44.7 us, 2 waves 42.7, 3 waves 53.0)
    int nw = static_cast<int>(((C < CW ? C : CW) + kClsPerWave - 1) / kClsPerWave);
    if (nw > 4) nw = 4;
    const int64_t fill = (fill_waves + G - 1) / G;
    if (nw > fill) nw = static_cast<int>(fill);
    p.nw = nw;
    // Few groups with many classes: one workgroup per group would leave most of the chip idle while each group walks
    // through its class tiles.  Then several workgroups share a group, each repeating the shared factorisation and
    // taking every splits-th tile, up to about 4096 waves in all.  From four tiles on: with fewer the repeated
    // factorisation and the extra launch cost what the split saves (G = 512, C = 100: 51 us whole, 59 us split).
    const int64_t tiles = (C + CW - 1) / CW;
    p.splits = 1;
    if (may_split && tiles >= 4) {
        const int64_t want = fill_waves / (G * nw);
        p.splits = static_cast<int>(want < tiles ? want : tiles);
        if (p.splits < 1) p.splits = 1;
    }
    return p;
}

struct GeneralShape {
    int cpw, nw, splits;
    size_t lds;                                            // 0: the shape does not fit the workgroup's LDS
};
GeneralShape general_shape(int64_t G, int K, int N, int n, int A, int64_t C, bool homogeneous, bool may_split) {
    GeneralShape s;
    const int KP = (K + 3) & ~3;
    const int M = K + A;
    // classes per wave: a class takes 2M lanes; waves per workgroup: enough for all classes, at most 4
    int cpw = kWave / (2 * M);
    if (cpw < 1) cpw = 1;
    if (cpw > C) cpw = static_cast<int>(C);
    const size_t fixed = sizeof(double) * (static_cast<size_t>(n - A) * KP + n + K + N) + sizeof(int) * (4 * static_cast<size_t>(N) + 2);
    const size_t per_class = sizeof(double) * (static_cast<size_t>(n) * (homogeneous ? 2 * M + 1 : 2 * M) + M + n);
    const size_t budget = 64 * 1024;
    while (cpw > 1 && fixed + cpw * per_class > budget) --cpw;
    const size_t per_wave = cpw * per_class;
    s.cpw = cpw;
    s.nw = 1;
    s.splits = 1;
    s.lds = 0;
    if (fixed + per_wave > budget) return s;
    int nw = static_cast<int>((C + cpw - 1) / cpw);
    if (nw > 4) nw = 4;
    if (nw > static_cast<int>((budget - fixed) / per_wave)) nw = static_cast<int>((budget - fixed) / per_wave);
    if (nw < 1) nw = 1;
    s.nw = nw;
    s.lds = fixed + nw * per_wave;
    // few groups, many classes: several workgroups share a group, as in the projected kernel (from four passes of a
    // workgroup over its classes on)
    const int64_t passes = (C + static_cast<int64_t>(nw) * cpw - 1) / (static_cast<int64_t>(nw) * cpw);
    if (may_split && passes >= 4) {
        const int64_t want = kFillWaves / (G * nw);
        s.splits = static_cast<int>(want < passes ? want : passes);
        if (s.splits < 1) s.splits = 1;
    }
    return s;
}

// most available workers a group can bring (S < 0: read off each mask)
int avail_capacity(int N, int S) { return S < 0 ? (N < APPROXIFER_MAX_AVAIL_BYZ ? N : APPROXIFER_MAX_AVAIL_BYZ) : N - S; }

int clear_workspace(int32_t *ws, int64_t G, int N, hipStream_t stream) {
    const int64_t words = G * (N + 1);
    const int threads = 256;
    return launch_status(launch_kernel(clear_workspace_kernel, dim3(static_cast<unsigned>((words + threads - 1) / threads)),
                                       dim3(threads), 0, stream, ws, words));
}

// Register tiles <rows of [V | I], rows of the projected system> of the projected kernel, smallest first.
struct ProjTile {
    int nb, rm;
};
constexpr ProjTile kProjTiles[] = {
    {20, 10},                 // n = 2M, the minimum of eq. (3), up to K + A = 10
    {20, 12}, {24, 12},       // n = 2M up to K + A = 12
    {24, 16}, {28, 14},       // n = 2M up to K + A = 14
    {32, 16}, {32, 32}, {48, 16}, {48, 32},
};
constexpr int kProjTileCount = sizeof(kProjTiles) / sizeof(kProjTiles[0]);
int proj_tile(int n, int M) {         // the smallest tile that holds (n, n - M); inside proj_domain one always does
    for (int t = 0; t < kProjTileCount; ++t)
        if (n <= kProjTiles[t].nb && n - M <= kProjTiles[t].rm) return t;
    return -1;
}
size_t basis_bytes(int tile, bool homogeneous) {
    const int stride = basis_stride(kProjTiles[tile].nb);
    const size_t b = sizeof(double) * (ush_rows(kProjTiles[tile].rm) * stride +
                                       (homogeneous ? kProjMaxM * stride + kProjMaxM * kProjMaxM : 0));
    return (b + 255) & ~static_cast<size_t>(255);
}
// Algorithm 1 on the shared factorisation: the register QR runs min(M, RM - 1) <= 15 steps.  Below K + A = 6 the LDS
// kernel, which packs 64 / 2M classes into a wave, is the faster one for many classes (measured, LDS / registers, 4096
// groups of 10 classes | 64 groups of 100: K + A = 3: 25 / 60 | 37 / 51 us; 5: 67 / 63 | 33 / 54; 6: 81 / 66 | 39 / 57;
// 8: 188 / 73 | 57 / 62; 10: 346 / 76 | 94 / 69; 14: 1275 / 111 | 201 / 97).
bool hom_proj_domain(int M, int n) { return proj_domain(M, n) && M >= 6 && M <= kProjMaxM - 1; }
size_t votes_bytes(int64_t G, int N) {
    return (sizeof(int32_t) * static_cast<size_t>(G) * (N + 1) + 255) & ~static_cast<size_t>(255);
}
// Groups with a full mask exist only when no fixed number of stragglers is asked for; the shared basis serves the
// projected kernel (Algorithm 2).
bool full_basis_applies(int N, int S, int M) { return S <= 0 && proj_domain(M, N); }

// The caller's workspace, carved: first the basis of the full node set (8-byte aligned), then the vote words.
struct Carved {
    double *basis;
    int32_t *votes;
};
Carved carve_workspace(void *d_workspace, size_t bytes, size_t need_basis, size_t need_votes) {
    Carved c = {nullptr, nullptr};
    unsigned char *p = static_cast<unsigned char *>(d_workspace);
    if (p == nullptr) return c;
    if (need_basis != 0 && reinterpret_cast<uintptr_t>(p) % sizeof(double) == 0 && bytes >= need_basis) {
        c.basis = reinterpret_cast<double *>(p);
        p += need_basis;
        bytes -= need_basis;
    }
    if (need_votes != 0 && reinterpret_cast<uintptr_t>(p) % sizeof(int32_t) == 0 && bytes >= need_votes)
        c.votes = reinterpret_cast<int32_t *>(p);
    return c;
}

// kNoFit: the shape does not fit this kernel's LDS (Algorithm 1 with many workers): the caller falls back.
constexpr int kNoFit = 1;

// Whether decode_byzantine_packed_kernel takes the call: one staged tile of fifteen class columns and the column of the
// denominators, and a factorisation of the workgroup's groups side by side (a row of U per lane of a 16-lane row) or, without
// stragglers, of one node set for all of them.  Its rows are workers, so that it works on rows of missing workers too: up
// to four more than the tile has it is the faster one throughout; with more, only Algorithm 2 from 2048 groups and tiles of
// 24 rows on (against a workgroup per group; K = 12, 28 of 46 workers, 4096 groups of 12 classes 69 and 86 us, Algorithm 1
// never: K = 10, 24 of 33, 650 and 577 us; K = 2, 6 of 26, 4096 groups, Algorithm 2: 36 and 25 us).
bool packed_domain(int NB, int RM, bool homogeneous, int64_t G, int N, int S, int M, int64_t C) {
    if (C > kClsLanes - 1 || M > kProjMaxM) return false;
    if (S == 0 && N <= NB && !homogeneous) return true;
    if (RM > kProjMaxM || N > 48) return false;
    return N <= NB + 4 || (!homogeneous && NB >= 24 && G > 2048);
}
// Groups per workgroup: one while the chip holds them all at once (five workgroups to each of 256 CUs), where spreading
// the classes over waves shortens the chain of a group; then as many as keep the launch at one round of workgroups.
// Measured with 1 / 2 / 4 groups, ten classes: K = 8, A = 2, 20 of 24 workers, 1024 groups 17.4 / 18.3 / 19.9 us, 2048
// groups 30.3 / 21.5 / 23.1 us, 4096 groups 52 / 37 / 30 us; K = 12, A = 2, 28 workers, 1024 groups 22.6 / 23.4 / 25.3
// us, 2048 groups 33 / 28 / 31 us, 8192 groups 87 / 74 / 68 us.  The lines lie right for 2, 5 and 15 classes too, but that
// two and five classes up to 1024 groups would be up to 13 % faster with two or four (K = 8, 2 classes, 1024 groups
// 15.4 / 15.0 / 14.0 us; 15 classes, 2048 groups 32 / 26 / 26).
// Algorithm 1's locator runs two waves to a SIMD: K = 8, 512 groups 31 / 33 / 43 us, 1024 groups 53 / 38 / 42 us, 2048
// groups 96 / 72 / 51 us; K = 12, 28 workers, 8192 groups 289 / 231 / 183 us.
int packed_groups(int64_t G, bool homogeneous) {
    if (homogeneous) return G <= 512 ? 1 : (G <= 1024 ? 2 : 4);
    return G <= 1280 ? 1 : (G <= 2560 ? 2 : 4);
}

// ---- two lanes to a class: the library's own nodes, few workers missing ------------------------------------------------
constexpr int kPairMostWorkers = 2 * 15 + 3 + kPairMaxMissing;            // of pair_shape

// cos(i pi / (N - 1)), N up to kPairMostWorkers; evaluated once, by the first call (N / 2 cosines took 0.2 us of each call's 2.3 on the host).
struct WorkerNodes {
    double x[kPairMostWorkers + 1][(kPairMostWorkers + 1) / 2];
    WorkerNodes() : x() {
        constexpr double kPi = 3.14159265358979323846;
        for (int N = 2; N <= kPairMostWorkers; ++N)
            for (int i = 0; 2 * i < N; ++i) x[N][i] = std::cos(i * kPi / (N - 1));
    }
};

// Whether the nodes are cos(i pi / (N - 1)) to a few roundings: the closed forms of locate_class_pair hold for these only.
bool chebyshev_workers(const Nodes &nodes, int N) {
    static const WorkerNodes table;
    constexpr double kClose = 16.0 / (1ull << 53);
    if (N > kPairMostWorkers) return false;
    for (int i = 0; 2 * i < N; ++i)
        if (!(std::fabs(nodes.beta[i] - table.x[N][i]) <= kClose) || !(std::fabs(nodes.beta[i] + nodes.beta[N - 1 - i]) <= kClose))
            return false;
    return true;
}

struct PairShape {
    int mt, tq;                                            // mt = 0: not for decode_byzantine_pairs_kernel
};
PairShape pair_shape(int K, int N, int S, int A, int64_t C, bool homogeneous) {
    const int M = K + A;
    // By the shape alone, never by the number of groups: the kernels round differently, and where fewer workers lie than A the
    // last bits decide who else goes, so that a group must not change kernels with the size of its call.  Where a line costs
    // small calls something the large ones decide: the chain of one wave is longer here than in the packed kernel, which gives a
    // group several waves.  Former kernels and this one, ten classes, 1 / 200 / 600 / 2000 groups, in us.  Algorithm 2, the far sizes:
    // K = 12, A = 3, 32 of 36 workers 23.4 / 24.0 / 33.9 / 75.3 and 27.2 / 27.7 / 27.5 / 30.1; K = 11, A = 2, 28 of 32 20.1 / 20.6 / 25.5 /
    // 46.3 and 21.9 / 22.3 / 22.3 / 24.4; K = 8, A = 1, 20 of 24 14.5 / 15.1 / 17.8 / 23.2 and 15.3 / 15.6 / 15.5 / 16.6.
    // Algorithm 1 adds rounds of inverse iteration, serial in the wave that has the slowest class: K = 10, A = 2, 24 of 28, a linear
    // model's answers 27.7 / 32.4 / 41.4 / 78.5 and 27.4 / 30.3 / 32.5 / 37.5, softmax answers 37 / 61 / 79 / 570 and 43 / 66 / 66 / 76; K = 11,
    // A = 2, 26 of 28, softmax 38 / 68 / 72 / 641 and 60 / 82 / 82 / 85.  It does not take wide tiles that leave their registers for scratch
    // and where A = 3 draws longer tails of rounds (the former kernels' time over this one's in 1600 drawn calls: A = 3 at K + A = 13
    // with S = 2 down to 0.76, at 14 from 0.85, 0.52 with S = 4; S > 2 at 14 at most 1.0; K + A = 15 0.22 to 2.3, mean 0.6).
    if (homogeneous && (M == 15 || (A == 3 && (M == 14 || (M == 13 && S > 1))) || (S > 2 && M == 14))) return {0, 0};
    if (S < 0 || S > kPairMaxMissing || M > 15 || A > kPairMaxAdversaries || C > (1 << 24)) return {0, 0};
    const int mt = std::max(4, (M + 1) & ~1), tq = std::max(mt / 2, (N - S - M + 1) / 2);
    if (tq > mt / 2 + 1 || 2 * tq - (N - S - M) > 1) return {0, 0};      // the latter: K = A = 1
    return {mt, tq};
}

// Whether a call of many classes that pair_shape takes has a use for votes' cells in the workspace: a workgroup to every 128 classes then,
// else one to a group that goes through them in turn.  Up to 512 groups, where one to each leaves places free (K = 8, A = 2, 20 of 24 workers, 300 of
// 1000 classes 86 us with and 111 without, 900 of 300 89 and 85), and for Algorithm 2 with K + A = 13 and 14 and nobody missing, where the
// split form alone has two waves to a SIMD (K = 12, A = 2, 513 groups of 130 55 and 81, 4000 of 130 282 and 418; K + A = 12: 224 and 177).
bool pair_votes(int64_t G, int M, int S, int64_t C, bool homogeneous) {
    return C > kPairClasses && (G <= 512 || (!homogeneous && S == 0 && (M == 13 || M == 14)));
}

// The rank-one term's inverse root for the rows of parity h: 1 + lift e e^T, e^T e = c, of the Gram matrix 1 - e e^T / (N - 1).
double pair_lift(int N, int R, int h) {
    const double c = h ? R / 2 : (R + 1) / 2 - 0.5;
    return (1.0 / std::sqrt(1.0 - c / (N - 1)) - 1.0) / c;
}

int run_pairs_shape(const PairShape &shape, const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_adv,
                    int32_t *d_status, int64_t G, int K, int N, int S, int A, int64_t C, bool vec4, const Nodes &nodes,
                    int sign_mode, bool homogeneous, int32_t *votes, hipStream_t stream) {
    PairCall call;
    call.preds = d_preds;
    call.mask = d_mask;
    call.out = d_out;
    call.adv = d_adv;
    call.status = d_status;
    call.votes = votes;
    call.G = G;
    call.C = C;
    call.K = K;
    call.N = N;
    call.S = S;
    call.A = A;
    call.sign_mode = sign_mode;
    call.lift0 = pair_lift(N, N - K - A, 0);
    call.lift1 = pair_lift(N, N - K - A, 1);
    call.gpw = 1;
    call.parts = call.splits = 1;
    call.vec4 = vec4;
    const int64_t Cv = vec4 ? C / 4 : C, tiles = (Cv + kColsPerTile - 1) / kColsPerTile;
    if (C > kPairClasses) {
        // more classes than a workgroup has pairs of lanes: a workgroup to every 128 of them, if there is a place for their votes
        call.parts = static_cast<int>((C + kPairClasses - 1) / kPairClasses);
        call.splits = votes != nullptr ? call.parts : 1;
        if (call.splits > 1) {
            if (G * std::max<int64_t>(call.splits, tiles) > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
            const int rc = clear_workspace(votes, G, N, stream);
            if (rc != APPROXIFER_OK) return rc;
        }
    } else {
        // as few groups to a workgroup as give every CU one, and no more than it has pairs for.  Ten classes, K = 8, A = 2, 20
        // of 24 workers, 4 / 8 / 12 groups: 1000 groups 13.3 / 13.5 / 14.0 us, 2048 groups 18.6 / 13.7 / 14.2, 3000 groups
        // 18.6 / 19.0 / 14.4; two classes, 8192 groups, 16 / 32 / 64 groups: 21 / 17.9 / 24 us.
        call.gpw = static_cast<int>(std::min<int64_t>((G + 255) / 256, kPairClasses / C));
    }
    const auto run = [&] {
        const auto of = [&](auto pairs, auto null_pairs) { return (homogeneous ? null_pairs : pairs)(shape.tq, call, nodes, stream); };
        switch (shape.mt) {
            case 4: return of(run_pairs_4, run_null_pairs_4);
            case 6: return of(run_pairs_6, run_null_pairs_6);
            case 8: return of(run_pairs_8, run_null_pairs_8);
            case 10: return of(run_pairs_10, run_null_pairs_10);
            case 12: return of(run_pairs_12, run_null_pairs_12);
            case 14: return of(run_pairs_14, run_null_pairs_14);
            default: return run_pairs_16(shape.tq, call, nodes, stream);      // Algorithm 2 only
        }
    };
    const int rc = run();
    if (rc != APPROXIFER_OK || call.splits == 1) return rc;
    return launch_status(launch_kernel(vec4 ? decode_located_kernel<4> : decode_located_kernel<1>, dim3(static_cast<unsigned>(G * tiles)),
                                       dim3(kPairThreads), located_lds_bytes(K, N, N - S - A), stream, d_preds, d_mask, votes, d_out,
                                       d_adv, d_status, K, N, S, A, C, Cv, tiles, sign_mode, nodes));
}

template <int NB, int RM, int NW, bool SHARED, bool HOMOG>
int run_packed_shape(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_adv, int32_t *d_status, int64_t G,
                     int K, int N, int S, int n, int A, int C, const Nodes &nodes, int sign_mode, const double *basis,
                     hipStream_t stream) {
    int gpw = packed_groups(G, HOMOG);
    // a wave per round of four classes, up to four, and one per group (five waves for the ten rounds of four groups
    // balance better and are slower from 4096 groups on, 100 us against 71 at K = 12, 8192 groups: fewer workgroups fit)
    const auto waves = [C](int groups) {
        const int rounds = (groups * C + kClsPerWave - 1) / kClsPerWave;
        return std::max(std::min(rounds, kPackedWaves), groups);
    };
    // two workgroups to a CU at least
    while (gpw > 1 && packed_lds_bytes<NB, RM, NW, HOMOG>(SHARED, gpw, waves(gpw), K + A) > kLdsPerCu / 2) gpw /= 2;
    const int nw = waves(gpw);
    const size_t lds = packed_lds_bytes<NB, RM, NW, HOMOG>(SHARED, gpw, nw, K + A);
    const auto kernel = decode_byzantine_packed_kernel<NB, RM, NW, SHARED, HOMOG>;
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(kernel, dim3(static_cast<unsigned>((G + gpw - 1) / gpw)), dim3(nw * kWave), lds, stream,
                                       d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n, A, C, sign_mode, gpw, basis,
                                       nodes));
}

// basis: the call's shared factorisation, or null.  S = 0 (a group whose mask is not full is bad then): all groups have it,
// whether it comes from the workspace or not, so that a workspace changes no bit.
template <int NB, int RM, bool HOMOG>
int run_packed(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_adv, int32_t *d_status, int64_t G,
               int K, int N, int S, int n, int A, int C, const Nodes &nodes, int sign_mode, const double *basis,
               hipStream_t stream) {
    if (S == 0)
        return run_packed_shape<NB, RM, NB, true, HOMOG>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n, A, C, nodes,
                                                         sign_mode, basis, stream);
    if constexpr (RM <= kProjMaxM) {
        if (N <= NB)
            return run_packed_shape<NB, RM, NB, false, HOMOG>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n, A, C, nodes,
                                                              sign_mode, nullptr, stream);
        if constexpr (NB < 48) {
            if (N <= NB + 4)
                return run_packed_shape<NB, RM, NB + 4, false, HOMOG>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n, A,
                                                                      C, nodes, sign_mode, nullptr, stream);
        }
        if constexpr (NB >= 24 && NB < 48 && !HOMOG)
            return run_packed_shape<NB, RM, 48, false, HOMOG>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n, A, C,
                                                              nodes, sign_mode, nullptr, stream);
    }
    return APPROXIFER_ERR_LIMIT;                          // not inside packed_domain
}

template <int NB, int RM, bool HOMOG>
int run_proj(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_adv, int32_t *d_status, int64_t G,
             int K, int N, int S, int A, int64_t C, int n_cap, bool vec4, const Nodes &nodes, int sign_mode,
             void *d_workspace, size_t workspace_bytes, int tile, hipStream_t stream) {
    const int KP = (K + 3) & ~3;
    const int M = K + A;
    const int64_t Cv = vec4 ? C / 4 : C;
    const size_t need_basis = full_basis_applies(N, S, M) ? basis_bytes(tile, HOMOG) : 0;
    const Carved ws = carve_workspace(d_workspace, workspace_bytes, need_basis, votes_bytes(G, N));
    // Algorithm 1's locator runs two waves to a SIMD (registers): half as many waves fill the chip
    ProjShape p = proj_shape(G, C, ws.votes != nullptr, HOMOG ? kFillWaves / 2 : kFillWaves);
    const int CW = 1 << p.cw_log2;
    const size_t hom_wave = HOMOG ? sizeof(double) * hom_scratch_doubles(M, NB, hom_mt(NB)) : 0;
    const size_t fixed = sizeof(double) * (static_cast<size_t>(basis_doubles<NB, RM, HOMOG>()) + (HOMOG ? kVDoubles - kVSquare : 0) +
                                           kPowers * lds_stride(NB) + NB +
                                           static_cast<size_t>(n_cap - A) * KP + K + N) +
                         sizeof(float) * (static_cast<size_t>(CW + 1) * y_stride(NB)) + sizeof(int) * (4 * static_cast<size_t>(N) + 2);
    constexpr size_t kBudget = kLdsPerCu / 2;              // two workgroups to a CU at least
    while (p.nw > 1 && fixed + p.nw * hom_wave > kBudget) --p.nw;
    const size_t lds = fixed + p.nw * hom_wave;
    if (lds > kBudget) return HOMOG ? kNoFit : APPROXIFER_ERR_LIMIT;   // Algorithm 2: cannot happen inside the domain
    if (G * p.splits > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const bool packed = packed_domain(NB, RM, HOMOG, G, N, S, M, C);
    if (ws.basis != nullptr && !(packed && S != 0)) {
        const hipError_t e = launch_kernel(full_basis_kernel<NB, RM, HOMOG>, dim3(1), dim3(kWave), 0, stream, ws.basis, N, M, nodes);
        if (e != hipSuccess) return APPROXIFER_ERR_LAUNCH;
    }
    if constexpr (RM <= kProjMaxM || !HOMOG) {
        if (packed)
            return run_packed<NB, RM, HOMOG>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, n_cap, A, static_cast<int>(C), nodes,
                                      sign_mode, S == 0 ? ws.basis : nullptr, stream);
    }
    if (p.splits > 1) {
        const int rc = clear_workspace(ws.votes, G, N, stream);
        if (rc != APPROXIFER_OK) return rc;
    }
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(decode_byzantine_proj_kernel<NB, RM, HOMOG>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    const dim3 grid(static_cast<unsigned>(G * p.splits)), block(p.nw * kWave);
    return launch_status(launch_kernel(decode_byzantine_proj_kernel<NB, RM, HOMOG>, grid, block, lds, stream, d_preds, d_mask, d_out,
                                       d_adv, d_status, K, N, S, A, C, Cv, vec4 ? 1 : 0, sign_mode, n_cap, p.cw_log2,
                                       p.splits, ws.votes, static_cast<const double *>(ws.basis), nodes));
}

}  // namespace

// Device address of this GPU's copy of the built-in workspace.  Looked up once per device, with that device current
// (every GPU has its own copy at its own address), and kept for the life of the process.
int static_workspace(void **d_ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static void *per_device[kMaxDevices] = {};
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return APPROXIFER_ERR_LAUNCH;
    std::lock_guard<std::mutex> hold(lock);
    if (per_device[device] == nullptr) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return APPROXIFER_ERR_LAUNCH;
        per_device[device] = p;
    }
    *d_ptr = per_device[device];
    return APPROXIFER_OK;
}

int launch_decode_rational(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_status, int64_t G, int K,
                           int N, int S, int A, int64_t C, const Nodes &nodes, hipStream_t stream) {
    const int n = avail_capacity(N, S);
    const int M = K + A;
    if (G > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    int cpw = kWave / (2 * M);
    if (cpw < 1) cpw = 1;
    if (cpw > C) cpw = static_cast<int>(C);
    const size_t fixed = sizeof(double) * (static_cast<size_t>(n) + K + N) + sizeof(int) * (static_cast<size_t>(N) + 2);
    const size_t per_class = sizeof(double) * (static_cast<size_t>(n) * 2 * M + M + n);
    const size_t budget = 64 * 1024;
    while (cpw > 1 && fixed + cpw * per_class > budget) --cpw;
    const size_t per_wave = cpw * per_class;
    if (fixed + per_wave > budget) return APPROXIFER_ERR_LIMIT;
    int nw = static_cast<int>((C + cpw - 1) / cpw);
    if (nw > 4) nw = 4;
    if (nw > static_cast<int>((budget - fixed) / per_wave)) nw = static_cast<int>((budget - fixed) / per_wave);
    if (nw < 1) nw = 1;
    return launch_status(launch_kernel(decode_rational_kernel, dim3(static_cast<unsigned>(G)), dim3(nw * kWave),
                                       fixed + nw * per_wave, stream, d_preds, d_mask, d_out, d_status, K, N, S, A, C, cpw, n,
                                       nodes));
}

size_t byzantine_workspace_bytes(int64_t G, int K, int N, int S, int A, int64_t C, bool pairs) {
    const int n = avail_capacity(N, S);
    const int M = K + A;
    bool splits = false;
    size_t basis = 0;
    if (proj_domain(M, n)) {
        splits = proj_shape(G, C, true).splits > 1;
        if (full_basis_applies(N, S, M)) basis = basis_bytes(proj_tile(n, M), hom_proj_domain(M, n));
    } else {
        splits = general_shape(G, K, N, n, A, C, false, true).splits > 1;
    }
    splits = splits || general_shape(G, K, N, n, A, C, true, true).splits > 1;       // Algorithm 1's locator
    // on the library's nodes, which this query is not told
    for (const bool homogeneous : {false, true})
        splits = splits || (pairs && pair_votes(G, M, S, C, homogeneous) && pair_shape(K, N, S, A, C, homogeneous).mt != 0);
    return basis + (splits ? votes_bytes(G, N) : 0);
}

int launch_decode_byzantine(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_adv,
                            int32_t *d_status, int64_t G, int K, int N, int S, int A, int64_t C, const Nodes &nodes,
                            int sign_mode, bool homogeneous, void *d_workspace, size_t workspace_bytes,
                            hipStream_t stream) {
    const int n = avail_capacity(N, S);
    const int M = K + A;
    const bool vec4 = (C % 4 == 0) && aligned16(d_preds) && aligned16(d_out);
    const int64_t Cv = vec4 ? C / 4 : C;
    if (G > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;

    const PairShape pair = pair_shape(K, N, S, A, C, homogeneous);
    if (pair.mt != 0 && chebyshev_workers(nodes, N)) {
        const Carved meet = carve_workspace(d_workspace, workspace_bytes, 0, pair_votes(G, M, S, C, homogeneous) ? votes_bytes(G, N) : 0);
        return run_pairs_shape(pair, d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, A, C, vec4, nodes, sign_mode, homogeneous,
                               meet.votes, stream);
    }
    if (homogeneous ? hom_proj_domain(M, n) : proj_domain(M, n)) {
        int rc = kNoFit;
#define APPROXIFER_PROJ(T, NB, RM)                                                                                     \
    case T:                                                                                                            \
        static_assert(kProjTiles[T].nb == NB && kProjTiles[T].rm == RM, "tile table");                                 \
        rc = homogeneous ? run_proj<NB, RM, true>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, A, C, n, vec4,     \
                                                  nodes, sign_mode, d_workspace, workspace_bytes, T, stream)            \
                         : run_proj<NB, RM, false>(d_preds, d_mask, d_out, d_adv, d_status, G, K, N, S, A, C, n, vec4,    \
                                                   nodes, sign_mode, d_workspace, workspace_bytes, T, stream);          \
        break;
        switch (proj_tile(n, M)) {
            APPROXIFER_PROJ(0, 20, 10)
            APPROXIFER_PROJ(1, 20, 12)
            APPROXIFER_PROJ(2, 24, 12)
            APPROXIFER_PROJ(3, 24, 16)
            APPROXIFER_PROJ(4, 28, 14)
            APPROXIFER_PROJ(5, 32, 16)
            APPROXIFER_PROJ(6, 32, 32)
            APPROXIFER_PROJ(7, 48, 16)
            APPROXIFER_PROJ(8, 48, 32)
            default: return APPROXIFER_ERR_LIMIT;          // cannot happen inside the projected kernel's domain
        }
#undef APPROXIFER_PROJ
        if (rc != kNoFit) return rc;
    }

    // the workgroups of a group meet in the workspace: without one that holds N + 1 words per group, and is aligned
    // for them, every group stays with one workgroup
    const Carved ws = carve_workspace(d_workspace, workspace_bytes, 0, votes_bytes(G, N));
    const GeneralShape sh = general_shape(G, K, N, n, A, C, homogeneous, ws.votes != nullptr);
    if (sh.lds == 0) return APPROXIFER_ERR_LIMIT;
    if (G * sh.splits > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    if (sh.splits > 1) {
        const int rc = clear_workspace(ws.votes, G, N, stream);
        if (rc != APPROXIFER_OK) return rc;
    }
    const dim3 grid(static_cast<unsigned>(G * sh.splits)), block(sh.nw * kWave);
    return launch_status(launch_kernel(homogeneous ? decode_byzantine_general_kernel<true> : decode_byzantine_general_kernel<false>,
                                       grid, block, sh.lds, stream, d_preds, d_mask, d_out, d_adv, d_status, K, N, S, A, C, Cv,
                                       vec4 ? 1 : 0, sign_mode, sh.cpw, n, sh.splits, ws.votes, nodes));
}

}  // namespace approxifer

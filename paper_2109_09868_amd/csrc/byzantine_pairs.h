// Algorithms 2 and 1 on the library's own worker nodes, beta_i = cos(i pi / (N - 1)), with at most four workers missing: two
// lanes to a class.
#pragma once

#include <type_traits>

#include "byzantine_general.h"
#include "rows.h"

namespace approxifer {

constexpr int kPairsPerWave = kWave / 2;
constexpr int kPairMaxAdversaries = 3;
constexpr int kPairMaxMissing = 4;
constexpr int kPairWaves = 4;                             // of a workgroup: one to a SIMD
constexpr int kPairThreads = kPairWaves * kWave, kPairRows = kPairThreads / 16;
constexpr int kPairClasses = kPairWaves * kPairsPerWave;  // of a workgroup

// Launch arguments of decode_byzantine_pairs_kernel, by value.
struct PairCall {
    const float *preds;
    const uint8_t *mask;
    float *out;
    int32_t *adv, *status, *votes;   // votes: the workspace, splits > 1
    int64_t G, C;
    int K, N, S, A, sign_mode;
    int gpw;                 // groups of a workgroup (whole groups), or
    int parts, splits;       // parts > 1: parts of a group's classes, each with a workgroup of its own (splits = parts) or one (1)
    bool vec4;               // as finish_group; parts > 1
    double lift0, lift1;     // see locate_class_pair
};

// A column whose square is below this part of the largest before it (Algorithm 1: of sum y^2) is rounding: it depends on the ones before it,
// as most do where only liars answer anything but zero or a constant.  The nodes are rational angles, so that such a column can also be
// zero to the last bit, or a rounding of roundings, and may not serve as a pivot next to others that are merely rounded.  K = 6, A = 1, 16
// workers, one liar's answers alone not zero: found in 0.79 of the classes without this, in all with it.  Liars' answers 1e14 times the others'
// are still found (both in numpy); honest float32 data leave nothing of use below 1e-14 of a column.
constexpr double kRoundingPart = 1e-28;

// x or y by a condition, as values: the compiler otherwise turns a choice between neighbouring elements of an array into
// one element at an address of its own, and keeps the array in memory for it.
__device__ __forceinline__ double choose(bool first, double x, double y) {
    asm("" : "+v"(x), "+v"(y));
    return first ? x : y;
}
__device__ __forceinline__ double pair_other(double v) { return dpp_exchange<kDppQuadXor1>(v); }
__device__ __forceinline__ int bits_of_other(unsigned mask) {             // ones in the other lane's mask
    return __builtin_amdgcn_update_dpp(0, static_cast<int>(__popc(mask)), kDppQuadXor1, 0xF, 0xF, true);
}
// v of this lane and of lane ^ DISTANCE, 16 or 32, added: the same bits in both
template <int DISTANCE>
__device__ __forceinline__ double rows_sum(double v) {
    const unsigned lo = __double2loint(v), hi = __double2hiint(v);
    if constexpr (DISTANCE == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    }
}
__device__ __forceinline__ double pair_sum(double v) { return v + pair_other(v); }
// minimum and maximum of numbers (no NaN): the plain instruction, without the quieting that fmin and fmax bring
__device__ __forceinline__ double min_number(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double min_magnitude(double a, double b) {    // min(|a|, b); b where a is not a number
    double r;
    asm("v_min_f64 %0, |%1|, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_number(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A double held in accumulation registers: the vector ALUs cannot read them, but they are there.
struct Parked {
    int lo, hi;
};
__device__ __forceinline__ Parked park(double v) {
    Parked p;
    asm("v_accvgpr_write_b32 %0, %1" : "=a"(p.lo) : "v"(__double2loint(v)));
    asm("v_accvgpr_write_b32 %0, %1" : "=a"(p.hi) : "v"(__double2hiint(v)));
    return p;
}
__device__ __forceinline__ double parked(const Parked &p) {
    int lo, hi;
    asm("v_accvgpr_read_b32 %0, %1" : "=v"(lo) : "a"(p.lo));
    asm("v_accvgpr_read_b32 %0, %1" : "=v"(hi) : "a"(p.hi));
    return __hiloint2double(hi, lo);
}

// Tile: MT >= M columns (even), S missing workers, TQ row slots to a lane: 2 TQ >= N - S - M > 2 TQ - 2.
template <int MT, int TQ, int S>
struct PairTile {
    static constexpr int kMH = MT / 2;
    static constexpr int TT = TQ + (S + 1) / 2;            // slots before the missing workers are taken out
    static constexpr int kLam = kMH + TT;                  // moments of one parity that the system is formed from
    static constexpr int kLamPad = (kLam + 1) & ~1;
    static constexpr int kNodes = (MT + 2 * TT + 1) / 2;   // most nodes that are not mirror images of others
    static constexpr int kTableDoubles = kNodes * 2 * kLamPad;
};

// The table tab[i][h][s] = w_i T_{2s+h}(beta_i) over the nodes i < ceil(N / 2), w_i = (-1)^i, halved at the end node and at
// a node in the middle (its own mirror image, which is counted twice); zero for i up to kNodes.  T_t(cos x) = cos t x: the
// values are nodes again.  A row of sixteen lanes takes every sixteenth t of sixteen nodes; `beta`: LDS.
template <int MT, int TQ, int S>
__device__ __forceinline__ void pair_table(double *tab, int N, const double *beta) {
    typedef PairTile<MT, TQ, S> Tile;
    constexpr int kTs = 2 * Tile::kLamPad;
    const int period = 2 * (N - 1), r = threadIdx.x / 16;
#pragma unroll
    for (int i0 = 0; i0 < Tile::kNodes; i0 += 16) {
        const int i = i0 + threadIdx.x % 16;
        const bool node = i < (N + 1) / 2;
        const double w = !node ? 0.0 : (i & 1 ? -1.0 : 1.0) * (i == 0 ? 0.5 : 1.0) * (2 * i == N - 1 ? 0.5 : 1.0);
        int step = node ? i * kPairRows : 0, k = node ? i * r : 0;       // modulo the period: i * 16 <= 4 periods
#pragma unroll
        for (int m = 4; m > 0; m /= 2) {
            step = step >= m * period ? step - m * period : step;
            k = k >= m * period ? k - m * period : k;
        }
#pragma unroll
        for (int t0 = 0; t0 < kTs; t0 += kPairRows) {
            const int t = t0 + r;
            const double v = beta[k < N ? k : period - k];
            if (i < Tile::kNodes && t < kTs) tab[i * kTs + (t & 1) * Tile::kLamPad + t / 2] = w * v;
            k += step;
            k = k >= period ? k - period : k;
        }
    }
}

// Algorithm 1 (HOMOG below): the unit vector (P, Q) of monomial coefficients that minimises sum_i (P(x_i) + y_i Q(x_i))^2 (the
// sign of y only flips that of Q), for the class of this pair of lanes.  With p, q the coefficients in the Chebyshev basis, D
// the matrix that takes them to monomials (T_e has terms of e's parity only, so it is a lane's own business), T the basis at
// the nodes that answered, G = T^T T and K = T^T diag(y) T, a round of the inverse iteration
//     [ G  K              ] [p']   [D^T D p]
//     [ K  T^T diag(y)^2 T ] [q'] = [D^T D q]
// is solved by eliminating p', which leaves B^T B for q', B the projected system of Algorithm 2 with all M columns, through its
// triangular factor (B is never squared):
//     u = G^-1 D^T D p,   B^T B q' = D^T D q - K u,   p' = u - G^-1 K q'.
// G^-1 is in closed form (diagonal and a rank-one term per parity, less the missing workers' rows), K's entries are sums of two
// moments as the system's are.  Start vector and settling rule are those of homogeneous_q, which is the fallback for a class that has not
// settled after kPairRounds; pivots of columns that depend on others are all raised to one floor, so that the null vector is a mixture of
// such columns (a single one has zeros at nodes of its own).
// Against the monomial QR (numpy, both): largest error of Q(x_i) relative to their maximum 1.6e-10 and 3e-8 at K = 12, A = 2,
// 28 workers, 3e-12 and 2e-11 at K = 8, A = 2, 20 of 24; the same number of rounds, two to four on rational data.
//   a: the system's columns (destroyed), k[s]: half the moment sum_i y_i T_{2s+h}(beta_i), square: sum_i y_i^2
//   c: coefficients of T_{2s+h} in Q.  Returns whether the class settled: the same in both lanes
constexpr int kPairRounds = 64;
// Rounds with a Ritz step, further and further apart: done often it keeps stirring up the third mode, and classes whose smallest
// singular values are within 5 % of each other never settle.  Of 550000 classes (six shapes; linear, ReLU and softmax answers and
// noise, liars or none; the iteration in numpy) all settle; every sixth round from the fifth on leaves 3 of them, every other
// round 1 of 8000.
constexpr unsigned long long kRitzRounds = 1ull << 1 | 1ull << 3 | 1ull << 5 | 1ull << 11 | 1ull << 19 | 1ull << 29 | 1ull << 41 | 1ull << 55;

// T_{2s+h} = sum_k c[h][k][s] x^{2k+h}
struct ChebyshevToMonomial {
    double c[2][8][8];
    constexpr ChebyshevToMonomial() : c() {
        double t[16][16] = {};
        t[0][0] = 1.0;
        t[1][1] = 1.0;
        for (int e = 2; e < 16; ++e)
            for (int d = 0; d <= e; ++d) t[e][d] = (d > 0 ? 2.0 * t[e - 1][d - 1] : 0.0) - t[e - 2][d];
        for (int h = 0; h < 2; ++h)
            for (int k = 0; k < 8; ++k)
                for (int s = 0; s < 8; ++s) c[h][k][s] = t[2 * s + h][2 * k + h];
    }
};
static __constant__ constexpr ChebyshevToMonomial kChebyshev;

template <int LANE>
__device__ __forceinline__ double pair_bcast(double v) {   // lane LANE of the pair's, to both
    return dpp_exchange<LANE == 0 ? 0xA0 : 0xF5>(v);      // quad_perm:[0,0,2,2], [1,1,3,3]
}

template <int MT, int TQ, int S>
__device__ __forceinline__ bool null_vector_pair(double (&a)[MT][TQ], const double (&k)[MT], double square, const double *own,
                                                 const double *basis, unsigned long long absent, int N, int M, int h, bool live,
                                                 double (&c)[MT / 2]) {
    constexpr int MH = MT / 2, kRow = 2 * PairTile<MT, TQ, S>::kLamPad;
    // ---- elimination, all columns in their order: nf as for Algorithm 2, rs[s] = 1 / pivot^2 of column 2s + h ---------------
    const double floor = kRoundingPart * square;
    const bool fits = square > 0.0 && square < __builtin_inf();
    double nf[MT][MH], rs[MH], even = 0.0;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        double r = 0.0;
        if (j < M) {
            double sig = a[j][0] * a[j][0];
#pragma unroll
            for (int t = 1; t < TQ; ++t) sig = fma(a[j][t], a[j][t], sig);
            sig = pair_sum(sig);
            r = rcp_normal(sig > floor ? sig : floor);    // the pivot; nothing is taken out along a column of rounding
            const double share = sig > floor ? r : 0.0;
            const auto take_out = [&](double (&to)[TQ]) {
                double d = a[j][0] * to[0];
#pragma unroll
                for (int t = 1; t < TQ; ++t) d = fma(a[j][t], to[t], d);
                const double f = -pair_sum(d) * share;
#pragma unroll
                for (int t = 0; t < TQ; ++t) to[t] = fma(f, a[j][t], to[t]);
                return f;
            };
#pragma unroll
            for (int s = (j + 1) / 2; s < MH; ++s) {
                double fe = 0.0;
                if (2 * s > j) fe = take_out(a[2 * s]);
                nf[j][s] = choose(h, take_out(a[2 * s + 1]), fe);
            }
        } else {
#pragma unroll
            for (int s = (j + 1) / 2; s < MH; ++s) nf[j][s] = 0.0;
        }
        r *= 2 * (N - 1);                                 // the rows of a[] are 2 ((N - 1) / 2)^1/2 times orthonormal ones'
        if (j % 2 == 0) even = r;
        else rs[j / 2] = choose(h, r, even);
    }
    const bool last = 2 * (MH - 1) + h < M;               // an odd M: lane 1 has no last entry

    // ---- G^-1 v = v / d - scale (sum v / d) / d + W W^T v -----------------------------------------------------------------
    const double over = 2.0 / (N - 1), over0 = h ? over : 0.5 * over;    // 1 / d_0, the others; d = 0 of no entry: none
    double inv[MH], sum_inv = 0.0;
#pragma unroll
    for (int s = 0; s < MH; ++s) {
        inv[s] = s == 0 ? over0 : (s < MH - 1 || last ? over : 0.0);
        sum_inv += inv[s];
    }
    const double scale = rcp_normal(1.0 + sum_inv);
    double w[S > 0 ? S : 1][MH];
    const auto full_inverse = [&](const double (&v)[MH], double (&to)[MH]) {
        double sum = 0.0;
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            to[s] = v[s] * inv[s];
            sum += to[s];
        }
        sum *= -scale;
#pragma unroll
        for (int s = 0; s < MH; ++s) to[s] = fma(sum, inv[s], to[s]);
    };
    const auto dot = [](const double (&v)[MH], const double (&z)[MH]) {
        double d = v[0] * z[0];
#pragma unroll
        for (int s = 1; s < MH; ++s) d = fma(v[s], z[s], d);
        return pair_sum(d);
    };
    const auto inverse = [&](const double (&v)[MH], double (&to)[MH]) {
        full_inverse(v, to);
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const double d = dot(w[b], v);
#pragma unroll
            for (int s = 0; s < MH; ++s) to[s] = fma(d, w[b][s], to[s]);
        }
    };
    if constexpr (S > 0) {                                // (G - X X^T)^-1 = G^-1 + W W^T, W = G^-1 X L^-T, L L^T = 1 - X^T G^-1 X
        double x[S][MH], l[S][S], rd[S];
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const int i0 = __builtin_ctzll(absent), i = 2 * i0 >= N ? N - 1 - i0 : i0;
            absent &= absent - 1ull;
            const double back = (i & 1 ? -1.0 : 1.0) * (i == 0 || 2 * i == N - 1 ? 2.0 : 1.0) * (2 * i0 >= N && h ? -1.0 : 1.0);
#pragma unroll
            for (int s = 0; s < MH; ++s) x[b][s] = s < MH - 1 || last ? back * own[i * kRow + s] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < S; ++b) {
            full_inverse(x[b], w[b]);
#pragma unroll
            for (int r = 0; r <= b; ++r) {
                l[b][r] = r < b ? 0.0 : 1.0;
                l[b][r] -= r < b ? dot(x[r], w[b]) : dot(x[b], w[b]);
            }
        }
        // rows of L in turn; w[b] becomes column b of W
#pragma unroll
        for (int b = 0; b < S; ++b) {
#pragma unroll
            for (int r = 0; r <= b; ++r) {
#pragma unroll
                for (int m = 0; m < r; ++m) l[b][r] = fma(-l[b][m], l[r][m], l[b][r]);
                if (r < b) l[b][r] *= rd[r];
            }
            rd[b] = rsqrt_normal(l[b][b]);
#pragma unroll
            for (int s = 0; s < MH; ++s) {
#pragma unroll
                for (int r = 0; r < b; ++r) w[b][s] = fma(-l[b][r], w[r][s], w[b][s]);
                w[b][s] *= rd[b];
            }
        }
    }

    // ---- K v: row 2t + h from own and the other lane's half moments, as the system's columns are formed ---------------------
    double ko[MT], below[MH], ahead[MT - 1];
#pragma unroll
    for (int s = 0; s < MT; ++s) ko[s] = pair_other(k[s]);
#pragma unroll
    for (int d = 1; d < MH; ++d) below[d] = choose(h, k[d - 1], k[d]);
#pragma unroll
    for (int s = 0; s < MT - 1; ++s) ahead[s] = choose(h, ko[s + 1], ko[s]);
    const auto multiply = [&](const double (&v)[MH], double (&to)[MH]) { // to -= K v
        double ve[MH], vo[MH];
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            ve[s] = -pair_bcast<0>(v[s]);
            vo[s] = -pair_bcast<1>(v[s]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < MH; ++t) {
            double sum = to[t];
#pragma unroll
            for (int u = 0; u < MH; ++u) {
                sum = fma(k[t + u], ve[u], sum);
                sum = fma(t >= u ? k[t >= u ? t - u : 0] : below[t >= u ? 1 : u - t], ve[u], sum);
                sum = fma(ahead[t + u], vo[u], sum);
                sum = fma(t > u ? ahead[t > u ? t - u - 1 : 0] : ko[t > u ? 0 : u - t], vo[u], sum);
            }
            to[t] = t < MH - 1 || last ? sum : 0.0;
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const double *mono = basis;
    // ---- inverse iteration; mp, mq: the monomial coefficients of the unit vector ----------------------------------------------
    const auto to_monomials = [&](const double (&v)[MH], double (&m)[MH]) {
#pragma unroll
        for (int d = 0; d < MH; ++d) {
            m[d] = 0.0;
#pragma unroll
            for (int s = d; s < MH; ++s) m[d] = fma(mono[d * MH + s], v[s], m[d]);
        }
    };
    const auto transposed = [&](const double (&m)[MH], double (&v)[MH]) {
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            v[s] = 0.0;
#pragma unroll
            for (int d = 0; d <= s; ++d) v[s] = fma(mono[d * MH + s], m[d], v[s]);
            if (s == MH - 1 && !last) v[s] = 0.0;
        }
    };
    double mp[MH], mq[MH];
#pragma unroll
    for (int s = 0; s < MH; ++s) {
        const bool in = s < MH - 1 || last;
        mp[s] = in ? 1.0 + 0.25 * ((2 * s + h) % 3) : 0.0;
        mq[s] = in ? 1.0 + 0.25 * ((M + 2 * s + h) % 3) : 0.0;
    }
    {
        double nn = 0.0;
#pragma unroll
        for (int s = 0; s < MH; ++s) nn = fma(mp[s], mp[s], fma(mq[s], mq[s], nn));
        const double unit = rsqrt_normal(pair_sum(nn));
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            mp[s] *= unit;
            mq[s] *= unit;
        }
    }
    double dd_prev = __builtin_inf(), ratio_before = dd_prev, quotient = 0.0;
    int since_jump = 0;
    bool settled = !fits;
    unsigned long long ritz = kRitzRounds;
    for (int round = 0; round < kPairRounds; ++round, ritz >>= 1) {
        // read again in every round: carried along it would take the registers that the rest of the round needs
        int offset = 0;
        asm volatile("" : "+v"(offset));
        mono = basis + offset;
        double f[MH], u[MH], t[MH];
        transposed(mp, f);
        __builtin_amdgcn_sched_barrier(0);
        inverse(f, u);
        __builtin_amdgcn_sched_barrier(0);
        transposed(mq, t);
        __builtin_amdgcn_sched_barrier(0);
        multiply(u, t);
        // (1 + N)^T, the pivots, (1 + N), N = -nf above the diagonal
#pragma unroll
        for (int j = 0; j < MT - 1; ++j) {
            const double tj = j % 2 == 0 ? pair_bcast<0>(t[j / 2]) : pair_bcast<1>(t[j / 2]);
#pragma unroll
            for (int s = (j + 1) / 2; s < MH; ++s) t[s] = fma(nf[j][s], tj, t[s]);
        }
        double part[MT];
#pragma unroll
        for (int j = 0; j < MT; ++j) part[j] = 0.0;
#pragma unroll
        for (int s = MH - 1; s >= 0; --s) {
            t[s] *= rs[s];
            const double odd = pair_sum(part[2 * s + 1]);
            part[2 * s] = fma(nf[2 * s][s], t[s] + odd, part[2 * s]);    // lane 1's; zero in lane 0
            c[s] = t[s] + choose(h, odd, pair_sum(part[2 * s]));
#pragma unroll
            for (int j = 0; j < 2 * s; ++j) part[j] = fma(nf[j][s], c[s], part[j]);
        }
#pragma unroll
        for (int s = 0; s < MH; ++s) f[s] = 0.0;
        multiply(c, f);
        inverse(f, t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < MH; ++s) u[s] += t[s];
        double np[MH], nq[MH];
        to_monomials(u, np);
        __builtin_amdgcn_sched_barrier(0);
        to_monomials(c, nq);
        __builtin_amdgcn_sched_barrier(0);
        double nn = 0.0;
#pragma unroll
        for (int s = 0; s < MH; ++s) nn = fma(np[s], np[s], fma(nq[s], nq[s], nn));
        const double unit = rsqrt_normal(pair_sum(nn));   // zero, inf or NaN: NaN, the class does not settle
        double dd = 0.0;
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            const double ep = fma(np[s], unit, -mp[s]), eq = fma(nq[s], unit, -mq[s]);   // z' . z > 0 always: no sign to align
            dd = fma(ep, ep, fma(eq, eq, dd));
        }
        dd = pair_sum(dd);
        const double dd_before = dd_prev;
        settled = settled || dd <= 1e-22 || (dd_prev <= 1e-16 && dd >= 0.25 * dd_prev);
        dd_prev = dd;
        ++since_jump;
        double old = 0.0, next = 1.0;                     // what of z and z' the next round starts from
        if (ritz & 2ull) {                                // in the next round
            quotient = round == 0 || dd > 1e-12 ? unit * fma(-0.5, dd, 1.0) : 0.0;   // z'^T A z', A z' = unit z
        } else if ((ritz & 1ull) && quotient > 0.0 && !settled && dd > (round == 1 ? 1e-18 : 1e-12) && dd < 1.0) {
            // The best vector of span(z, z') while the steps are large: where two modes are left the slow one is gone with it, also
            // where the iterate still lies by the wrong one of them (half < 0).
            const double g = fma(-0.5, dd, 1.0), across2 = dd * fma(-0.25, dd, 1.0), across = sqrt_normal(across2);
            const double r = rcp_normal(across), mixed = fma(-g, quotient, unit) * r, other = g * fma(g, quotient, -unit) * r * r;
            const double half = 0.5 * (other - quotient), root = fabs(half) + sqrt_normal(fma(half, half, mixed * mixed));
            const double norm = rsqrt_normal(fma(root, root, mixed * mixed));          // of (root, -mixed) or (-mixed, root)
            const double along = (half > 0.0 ? root : -mixed) * norm, tau = (half > 0.0 ? -mixed : root) * norm * r;
            if (tau > 0.0) {
                old = fma(-tau, g, along);
                next = tau;
                if (!(next > 0.95 && next < 1.05)) dd_prev = __builtin_inf();
            }
        }
        // A slow decay is followed to its limit once it is steady: two ratios of successive steps that differ by a tenth of their
        // distance from 1 (a third mode that still decays makes them differ, and the jump would bring it back).
        double ratio = __builtin_inf();
        if (round > 1 && !settled && dd <= 1e-10 && dd_before < __builtin_inf()) {
            ratio = sqrt_normal(dd * rcp_normal(dd_before));
            if (since_jump >= 3 && ratio > 0.05 && ratio < 0.9995 && fabs(ratio - ratio_before) <= 0.1 * (1.0 - ratio)) {
                old = -ratio * rcp_normal(1.0 - ratio);
                next = 1.0 - old;
                since_jump = 0;
                dd_prev = __builtin_inf();
            }
        }
        ratio_before = ratio;
        if (settled) {                                    // it stays: how often the wave's other classes still go round is not to show
            old = 1.0;
            next = 0.0;
        }
#pragma unroll
        for (int s = 0; s < MH; ++s) {
            mp[s] = fma(old, mp[s], next * unit * np[s]);
            mq[s] = fma(old, mq[s], next * unit * nq[s]);
        }
        if (__all((settled || !live) ? 1 : 0)) break;
    }
    // No fit: an answer that is not a number, or zeros throughout.  Equal magnitudes, as from the Jacobi iteration of such a class, which
    // takes a wave for it alone (one worker's NaN in every class of 2048 groups, K = 8, A = 2, 20 of 24 workers: 5.5 ms, 19 us this way).
#pragma unroll
    for (int s = 0; s < MH; ++s) c[s] = fits ? c[s] : __builtin_nan("");
    return settled;
}

// Algorithm 2 (HOMOG: Algorithm 1), steps 1-5, for the class of this pair of lanes; h = lane % 2.
//
// The polynomial P is eliminated in closed form.  With omega = (1/2, 1, .., 1, 1/2) the Chebyshev polynomials are orthogonal
// on the nodes, so the rows u_r = omega T_{N-1-r} = w T_r, r < R = N - M, are orthogonal to every polynomial of degree
// below M; their Gram matrix in the plain inner product is diagonal but for -1/2 between rows of equal parity, a rank-one
// term for either parity, whose inverse root (1 + lift e e^T per parity, e_0 = sqrt(1/2), else 1) makes them orthonormal.
// In the same basis for Q the system's entries are sums of two moments,
//     u_r diag(y) T_e = (lambda_{r+e} + lambda_|r-e|) / 2,     lambda_t = sum_i w_i y_i T_t(beta_i),
// and the mirror images beta_{N-1-i} = -beta_i halve the work for the moments: no factorisation of the nodes, and a sixth
// of the multiply-adds of forming U diag(y) V entry by entry.  A missing worker's prediction counts as a free unknown (its
// column u_r e_i is reflected out ahead, y_i = 0).  Q_0 = 1 is sum_e q_e T_e(0) = 1, which takes the even
// columns to T_e - T_e(0).
// Rows of parity h live in lane h (row 2t + h in slot t): the moments of a parity, the rank-one term and the even and odd
// part of Q are a lane's own, and a dot product over the rows is two short ones and an exchange.  The elimination is
// modified Gram-Schmidt on [columns 1 .. M-1 | column 0], with the right-hand side carried along as backward stable as
// reflections (Bjorck 1967).  Next to the monomial basis its solutions are closer to the exact
// ones: largest error of Q(x_i) relative to their maximum over 60 draws (both forms in numpy), K = 12, A = 2, 28 workers 2e-9 and 2e-8, K = 8, A =
// 2, 20 of 24 workers 1.4e-10 and 5e-10.
//   y, ys: the class's predictions, y[i ys] for worker i (LDS), zero where there is no answer
//   bits: workers that answered, missing: the others;  votes: the group's counters;  live: the pair has a class
// Returns whether the class has voted (Algorithm 1 may not have settled).
template <int MT, int TQ, int S, bool HOMOG>
__device__ __forceinline__ bool locate_class_pair(const float *y, int ys, unsigned long long bits, unsigned long long missing,
                                                  const double *tab, const double *mono, int N, int M, int A, int h, double lift,
                                                  bool live, int *votes) {
    typedef PairTile<MT, TQ, S> Tile;
    typedef double v2d __attribute__((ext_vector_type(2)));
    constexpr int TT = Tile::TT, MH = Tile::kMH, kLam = Tile::kLam, kRow = 2 * Tile::kLamPad;
    const int NH = (N + 1) / 2;
    const int R = N - M;
    const double mirror = ((N - 1 + h) & 1) ? -1.0 : 1.0;  // w_{N-1-i} T_t(beta_{N-1-i}) against node i, t of parity h
    const double *own = tab + h * Tile::kLamPad;

    const unsigned long long absent = missing;

    // ---- moments: p[s] = lambda_{2s+h}, o[s] = lambda_{2s+1-h} -----------------------------------------------------------
    double p[Tile::kLamPad];
#pragma unroll
    for (int s = 0; s < Tile::kLamPad; ++s) p[s] = 0.0;
    double k[HOMOG ? MT : 1], square = 0.0;               // HOMOG: k[s] = sum_i y_i T_{2s+h}(beta_i) / 2; sum y^2
#pragma unroll
    for (int s = 0; s < (HOMOG ? MT : 1); ++s) k[s] = 0.0;
    {
        // a node's row is read while the one before it is multiplied: left to itself the compiler waits for every two reads
        constexpr int kReads = Tile::kLamPad / 2;
        v2d row[2][kReads];
        float lo[2], hi[2];
        const auto read = [&](int i) {
#pragma unroll
            for (int s = 0; s < kReads; ++s) row[i & 1][s] = *reinterpret_cast<const v2d *>(own + i * kRow + 2 * s);
            lo[i & 1] = y[i * ys];
            hi[i & 1] = y[(N - 1 - i) * ys];
        };
        read(0);
#pragma unroll
        for (int i = 0; i < Tile::kNodes; ++i) {          // N >= kNodes; rows past NH of the table are zero
            if (i + 1 < Tile::kNodes) read(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            const double near = lo[i & 1], far = hi[i & 1];
            const double z = fma(mirror, far, near);
#pragma unroll
            for (int s = 0; s < kReads; ++s) {
                p[2 * s] = fma(row[i & 1][s][0], z, p[2 * s]);
                p[2 * s + 1] = fma(row[i & 1][s][1], z, p[2 * s + 1]);
            }
            if constexpr (HOMOG) {
                const double v = (i & 1 ? -0.5 : 0.5) * (i == 0 ? 2.0 : 1.0) * fma(h ? -1.0 : 1.0, far, near);
#pragma unroll
                for (int s = 0; s < MT; ++s) k[s] = fma(row[i & 1][s / 2][s % 2], v, k[s]);
                square = fma(near, near, fma(far, far, square));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (HOMOG) {                                // here and not where they are used, with the table's rows kept until then
#pragma unroll
        for (int s = 0; s < MT; ++s) asm volatile("" : "+v"(k[s]));
        asm volatile("" : "+v"(square));
    }
    double o[kLam], below[MH], ahead[kLam - 1];
#pragma unroll
    for (int s = 0; s < kLam; ++s) o[s] = pair_other(p[s]);
#pragma unroll
    for (int d = 1; d < MH; ++d) below[d] = choose(h, p[d - 1], p[d]);       // lambda_{|h - 2d|}
#pragma unroll
    for (int s = 0; s < kLam - 1; ++s) ahead[s] = choose(h, o[s + 1], o[s]); // lambda_{2s+1+h}

    // ---- the system: a[e][t] = entry (2t + h, e), orthonormal rows, without the span of the missing workers' columns ------
    const double first = h ? 1.0 : 0.70710678118654752440;              // sqrt(1/2) for row 0
    double there[2];                                      // 2t + h < R for the last two slots
#pragma unroll
    for (int t = TT - 2; t < TT; ++t) there[t - TT + 2] = 2 * t + h < R ? 1.0 : 0.0;
    const auto orthonormal = [&](double (&c)[TT]) {
        c[0] *= first;
        c[TT - 2] *= there[0];
        c[TT - 1] *= there[1];
        double sum = first * c[0];
#pragma unroll
        for (int t = 1; t < TT; ++t) sum += c[t];
        sum *= lift;
        c[0] = fma(TT == 2 ? first * there[0] : first, sum, c[0]);
#pragma unroll
        for (int t = 1; t < TT; ++t) c[t] = t < TT - 2 ? c[t] + sum : fma(there[t - TT + 2], sum, c[t]);
    };
    // Reflections that take the missing workers' columns to the last S rows; the rows before these are then free of them.
    double x[S > 0 ? S : 1][TT], scale[S > 0 ? S : 1];
    const auto reflect = [&](double (&c)[TT], int s) {
        double d = x[s][0] * c[0];
#pragma unroll
        for (int t = 1; t < TT; ++t) d = fma(x[s][t], c[t], d);
        const double f = pair_sum(d) * scale[s];
#pragma unroll
        for (int t = 0; t < TT; ++t) c[t] = fma(f, x[s][t], c[t]);
    };
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int w = __builtin_ctzll(missing);
        missing &= missing - 1ull;
        const double sign = 2 * w >= N ? mirror : 1.0;
        const double *row = own + (2 * w >= N ? N - 1 - w : w) * kRow;
#pragma unroll
        for (int t = 0; t < TT; ++t) x[s][t] = sign * row[t];
    }
#pragma unroll
    for (int s = 0; s < S; ++s) orthonormal(x[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int r = R - 1 - s;
        double sig = 0.0, at = 0.0;                       // over the rows up to r; row r itself.  R >= 2 TT - 2
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            if (2 * t + 1 >= 2 * TT - 3 - s) {
                x[s][t] = 2 * t + h <= r ? x[s][t] : 0.0;
                at = 2 * t + h == r ? x[s][t] : at;
            }
            sig = fma(x[s][t], x[s][t], sig);
        }
        sig = pair_sum(sig);
        at = pair_sum(at);
        const double norm = sqrt_normal(sig), to = at >= 0.0 ? -norm : norm;
        scale[s] = -rcp_normal(fma(-to, at, sig));
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (2 * t + 1 >= 2 * TT - 3 - s) x[s][t] = 2 * t + h == r ? x[s][t] - to : x[s][t];
#pragma unroll
        for (int b = s + 1; b < S; ++b) reflect(x[b], s);
    }
    double a[MT][TQ];
    const double kept = 2 * (TQ - 1) + h < R - S ? 1.0 : 0.0;
    const auto column = [&](double (&c)[TT], double (&to)[TQ]) {
        orthonormal(c);
#pragma unroll
        for (int s = 0; s < S; ++s) reflect(c, s);
#pragma unroll
        for (int t = 0; t < TQ; ++t) to[t] = S > 0 && t == TQ - 1 ? kept * c[t] : c[t];
    };
    // odd columns first: the other lane's moments are then done with
    constexpr bool kPark = MT * TQ + S * TT > 130;        // .. and their columns out of the way, where registers are short
    Parked away[MH][TQ];
#pragma unroll
    for (int u = 0; u < MH; ++u) {
        double c[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) c[t] = ahead[t + u] + (t > u ? ahead[t > u ? t - u - 1 : 0] : o[t > u ? 0 : u - t]);
        column(c, a[2 * u + 1]);
        if constexpr (kPark) {
#pragma unroll
            for (int t = 0; t < TQ; ++t) away[u][t] = park(a[2 * u + 1][t]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < MH; ++u) {
        double c[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) c[t] = p[t + u] + (t >= u ? p[t >= u ? t - u : 0] : below[t >= u ? 1 : u - t]);
        column(c, a[2 * u]);
        if (!HOMOG && u > 0) {
#pragma unroll
            for (int t = 0; t < TQ; ++t) a[2 * u][t] += u % 2 ? a[0][t] : -a[0][t];      // T_{2u}(0) = (-1)^u
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    if constexpr (kPark) {
#pragma unroll
        for (int u = 0; u < MH; ++u)
#pragma unroll
            for (int t = 0; t < TQ; ++t) a[2 * u + 1][t] = parked(away[u][t]);
    }

    double c[MH];                                         // c[s]: coefficient of T_{2s+h} in Q
    bool settled = true;
    if constexpr (HOMOG) {
        settled = null_vector_pair<MT, TQ, S>(a, k, square, own, mono, absent, N, M, h, live, c);
    } else {
        // ---- elimination: nf[j][e / 2] = minus the share of column j in column e, lane e % 2 keeping it ------------------------
        double nf[MT][MH], most = 0.0;                        // the largest sig so far
    #pragma unroll
        for (int j = 1; j < MT; ++j) {
            if (j < M) {
                double sig = a[j][0] * a[j][0];
    #pragma unroll
                for (int t = 1; t < TQ; ++t) sig = fma(a[j][t], a[j][t], sig);
                sig = pair_sum(sig);
                most = max_number(most, sig);
                const double rs = sig > kRoundingPart * most ? rcp_normal(sig) : 0.0;      // a column of rounding: coefficient zero
                const auto take_out = [&](double (&c)[TQ]) {
                    double d = a[j][0] * c[0];
    #pragma unroll
                    for (int t = 1; t < TQ; ++t) d = fma(a[j][t], c[t], d);
                    const double f = -pair_sum(d) * rs;
                    if (j + 1 < MT) {                         // the right-hand side's remainder is not needed at the end
    #pragma unroll
                        for (int t = 0; t < TQ; ++t) c[t] = fma(f, a[j][t], c[t]);
                    }
                    return f;
                };
                nf[j][0] = choose(h, 0.0, take_out(a[0]));
    #pragma unroll
                for (int s = (j + 1) / 2; s < MH; ++s) {      // columns 2s (if behind j) and 2s + 1
                    double fe = 0.0;
                    if (2 * s > j) fe = take_out(a[2 * s]);
                    nf[j][s] = choose(h, take_out(a[2 * s + 1]), fe);
                }
            } else {
    #pragma unroll
                for (int s = 0; s < MH; ++s) nf[j][s] = 0.0;
            }
        }

        // ---- back substitution: c[s] = coefficient of T_{2s+h} in Q ---------------------------------------------------------------
        double part[MT];
    #pragma unroll
        for (int j = 1; j < MT; ++j) part[j] = nf[j][0];
        double q0 = 1.0;
    #pragma unroll
        for (int s = MH - 1; s >= 0; --s) {
            const double qo = 2 * s + 1 < M ? pair_sum(part[2 * s + 1]) : 0.0;
            double qe = 0.0;
            if (s > 0) {
                part[2 * s] = fma(nf[2 * s][s], qo, part[2 * s]);            // lane 1's; zero in lane 0
                qe = 2 * s < M ? pair_sum(part[2 * s]) : 0.0;
                q0 += s % 2 ? qe : -qe;                       // Q_0 = 1: minus T_{2s}(0) of every even column
            }
            c[s] = h ? qo : (s > 0 ? qe : q0);
    #pragma unroll
            for (int j = 1; j < 2 * s; ++j) part[j] = fma(nf[j][s], c[s], part[j]);
        }
    }

    // ---- a_i = Q(beta_i), up to sign: lane 0 node i, lane 1 its mirror image; the A smallest vote --------------------------
    // A lane keeps its magnitudes and its three smallest; with the other lane's these give the A-th smallest of all, and who is
    // not above it votes.  All bits of a magnitude count: of equal ones alone the smaller worker index comes first.
    const unsigned answered = static_cast<unsigned>(h ? __brevll(bits) >> (64 - N) : bits);
    const unsigned mine = answered & ((1u << (h ? N / 2 : NH)) - 1u);    // bit i: this lane's node i; a middle one is lane 0's
    double size[Tile::kNodes];
    double l0 = __builtin_inf(), l1 = __builtin_inf(), l2 = __builtin_inf();
    {
        const double side = h ? -1.0 : 1.0;
        constexpr int kReads = (MH + 1) / 2, kAhead = 2;  // rows are read two nodes ahead
        v2d row[kAhead + 1][kReads];
        const auto read = [&](int i) {
#pragma unroll
            for (int s = 0; s < kReads; ++s) row[i % (kAhead + 1)][s] = *reinterpret_cast<const v2d *>(own + i * kRow + 2 * s);
        };
#pragma unroll
        for (int i = 0; i < kAhead && i < Tile::kNodes; ++i) read(i);
#pragma unroll
        for (int i = 0; i < Tile::kNodes; ++i) {
            if (i + kAhead < Tile::kNodes) read(i + kAhead);
            __builtin_amdgcn_sched_barrier(0);
            double v = 0.0;
#pragma unroll
            for (int s = 0; s < MH; ++s) v = fma(row[i % (kAhead + 1)][s / 2][s % 2], c[s], v);
            v = fma(side, pair_other(v), v);
            if (i == 0) v += v;                           // the table has half of these
            if (i >= Tile::kNodes - 4 && 2 * i == N - 1) v += v;
            v = min_magnitude(v, __builtin_inf());        // not a number: behind every number
            // nor does a worker that did not answer, or a row past the last node, come before any that did
            const bool there = S > 0 ? (mine & (1u << i)) != 0u : i < Tile::kNodes - 4 || (i < NH && !(h && 2 * i == N - 1));
            v = there ? v : __builtin_inf();
            size[i] = v;
            l2 = min_number(l2, max_number(l1, v));
            l1 = min_number(l1, max_number(l0, v));
            l0 = min_number(l0, v);
        }
    }
    const double m0 = pair_other(l0), m1 = pair_other(l1), m2 = pair_other(l2);
    const double last = A == 1 ? min_number(l0, m0)
                               : (A == 2 ? min_number(min_number(l1, m1), max_number(l0, m0))
                                         : min_number(min_number(l2, m2), min_number(max_number(l0, m1), max_number(l1, m0))));
    unsigned picks = 0u;
#pragma unroll
    for (int i = 0; i < Tile::kNodes; ++i) picks |= size[i] <= last ? 1u << i : 0u;
    picks &= mine;
    if (static_cast<int>(__popc(picks)) + bits_of_other(picks) > A) {   // of those that equal the A-th the first workers, lane 0's in ascending order
        unsigned less = 0u;
#pragma unroll
        for (int i = 0; i < Tile::kNodes; ++i) less |= size[i] < last ? 1u << i : 0u;
        less &= mine;
        unsigned equal = picks & ~less;
        const int ahead = bits_of_other(equal);           // both lanes are here: the sum above is the same in either
        int room = A - static_cast<int>(__popc(less)) - bits_of_other(less) - (h ? ahead : 0);
        picks = less;
        for (; room > 0 && equal != 0u; --room) {
            const unsigned next = h ? 1u << (31 - __builtin_clz(equal)) : equal & -equal;
            picks |= next;
            equal &= ~next;
        }
    }
    if (live && settled) {
        for (; picks != 0u; picks &= picks - 1u) {
            const int i = __builtin_ctz(picks);
            atomicAdd(&votes[h ? N - 1 - i : i], 1);
        }
    }
    return settled;
}

// The A most voted workers (equal counts: smaller index first), a lane to a worker (N < 64): bit w is worker w.  By a whole wave.
__device__ __forceinline__ unsigned long long most_voted(const int *votes, int N, int A) {
    const int lane = lane_id();
    int key = lane < N ? (votes[lane] << 6) | (kWave - 1 - lane) : -1;
    unsigned long long drop = 0ull;
    for (int pick = 0; pick < A; ++pick) {
        int m = key;
        m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor1, 0xF, 0xF, true));
        m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor2, 0xF, 0xF, true));
        m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowHalfMirror, 0xF, 0xF, true));
        m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowMirror, 0xF, 0xF, true));
        m = max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
                max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
        drop |= 1ull << (kWave - 1 - (m & (kWave - 1)));
        key = key == m ? -1 : key;
    }
    return drop;
}

// The decoder contraction of one group by a workgroup of few waves: a wave takes all queries of 64 vector columns, so that it reads every row
// once, and the next rows are on their way while it multiplies the last ones.
template <int VEC, int QUADS>
__device__ __forceinline__ void contract_columns(const float *__restrict__ pg, float *__restrict__ og, const int *F, int nF, int K, int KP,
                                                 int64_t C, int64_t Cv, const double *WdT) {
    typedef typename PredVec<VEC>::type V;
    for (int64_t cv = static_cast<int64_t>(wave_id()) * kColsPerTile + lane_id(); cv < Cv; cv += kPairWaves * kColsPerTile) {
        double acc[4 * QUADS][VEC];
#pragma unroll
        for (int j = 0; j < 4 * QUADS; ++j)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[j][e] = 0.0;
        V ahead[kRowChunk];
        load_row_chunk<VEC>(pg, F, nF, 0, C, cv, ahead);
        for (int r0 = 0; r0 < nF; r0 += kRowChunk) {
            V y[kRowChunk];
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u) y[u] = ahead[u];
            if (r0 + kRowChunk < nF) load_row_chunk<VEC>(pg, F, nF, r0 + kRowChunk, C, cv, ahead);
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u) {
                if (r0 + u < nF) {
#pragma unroll
                    for (int q = 0; q < QUADS; ++q) {
                        if (4 * q < KP) {
                            const double *w = WdT + (r0 + u) * KP + 4 * q;
#pragma unroll
                            for (int j = 0; j < 4; ++j)
#pragma unroll
                                for (int e = 0; e < VEC; ++e)
                                    acc[4 * q + j][e] = fma(w[j], static_cast<double>(vec_get<VEC>(y[u], e)), acc[4 * q + j][e]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4 * QUADS; ++j)
            if (j < K) store_row<VEC>(og + static_cast<size_t>(j) * C + cv * VEC, acc[j]);
    }
}

// A workgroup takes `gpw` whole groups (C <= 128), a class to a pair of lanes, and decodes them, a row
// of sixteen lanes to sixteen classes of a group:
//     out[j][c] = (sum_i T[j][i] s_i y_ic) / (sum_i T[j][i] s_i),     T[j][i] = 1 / (alpha_j - beta_i),
// lane j of the row holding T[j][i], which reaches the classes inside the multiply-add and sums the denominator of query j;
// s_i is the sign of worker i, 0 if it does not count.  A query node that is a worker's node has T = 0 there and takes that
// worker's row.  More classes: a workgroup to every 128 of a group's (kPart) that leaves its votes in the workspace, from where
// decode_located_kernel goes on: that launch alone writes outputs, so that one which fails leaves all of them as they were.  Without a
// workspace one workgroup takes all classes in turn (kParts: the loop costs 50 registers, and with them the second wave of a SIMD) and
// decodes its group itself.  No row of a worker that did not answer is read.
// dynamic LDS: double tab | beta_s[N] | whole groups: T[N][16] | sgn[16][N]
//              | float Ysh[groups][N][classes] | uint64 bits[gpw] | int votes[gpw][64] | hit[16]
//              | HOMOG: double mono[2][MT / 2][MT / 2] | scratch[4][pair_scratch_doubles]
__host__ __device__ constexpr int pair_decode_doubles(bool whole, int N) {
    const int d = whole ? 16 * N + kPairRows * N + N : N;
    return (d + 1) & ~1;
}
__host__ __device__ constexpr int64_t pair_tile_floats(bool whole, int gpw, int N, int64_t C) {
    return ((whole ? gpw * N * C : static_cast<int64_t>(N) * kPairClasses) + 3) & ~static_cast<int64_t>(3);
}
__host__ __device__ constexpr int pair_scratch_doubles(int N, int n, int M) {     // of a wave (HOMOG): xs, see locate_classes_wave, avail
    return N + n * (2 * M + 1) + M + n + (N + 1) / 2;
}
template <int MT, int TQ, int S>
constexpr size_t pair_lds_bytes(bool whole, int gpw, int N, int M, int64_t C, bool homogeneous) {
    return sizeof(double) * (PairTile<MT, TQ, S>::kTableDoubles + pair_decode_doubles(whole, N)) +
           sizeof(float) * pair_tile_floats(whole, gpw, N, C) + sizeof(uint64_t) * gpw + sizeof(int) * (kWave * gpw + 16) +
           (homogeneous ? sizeof(double) * (MT * MT / 2 + kPairWaves * pair_scratch_doubles(N, N - S, M)) : 0);
}

enum PairMode { kWhole, kPart, kParts };

template <int MT, int TQ, int S, PairMode MODE, bool HOMOG>
constexpr int kPairWavesPerSimd = MT * TQ + S * (TQ + (S + 1) / 2) + (HOMOG ? 2 * MT : 0) <= (MODE == kParts ? 60 : 100) ? 2 : 1;

template <int MT, int TQ, int S, PairMode MODE, bool HOMOG>
__global__ __launch_bounds__(kPairThreads) __attribute__((amdgpu_waves_per_eu(kPairWavesPerSimd<MT, TQ, S, MODE, HOMOG>))) void decode_byzantine_pairs_kernel(
    const PairCall a, const Nodes nodes) {
    typedef PairTile<MT, TQ, S> Tile;
    extern __shared__ __align__(16) double lds_d[];
    constexpr bool whole = MODE == kWhole;
    const int K = a.K, N = a.N, A = a.A, M = K + A;
    const int tid = threadIdx.x, wv = wave_id(), lane = lane_id(), h = lane & 1;
    double *tab = lds_d;
    double *beta_s = tab + Tile::kTableDoubles;
    double *T = beta_s + N;
    double *sgn = T + 16 * N;
    float *Ysh = reinterpret_cast<float *>(beta_s + pair_decode_doubles(whole, N));
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(Ysh + pair_tile_floats(whole, a.gpw, N, a.C));
    int *votes = reinterpret_cast<int *>(bits + a.gpw);
    int *hit = votes + kWave * a.gpw;
    // HOMOG: the basis change, and a scratch for each wave's classes that do not settle
    double *mono = reinterpret_cast<double *>(hit + 16);
    double *scratch = mono + 2 * Tile::kMH * Tile::kMH;

    const int64_t g0 = whole ? static_cast<int64_t>(blockIdx.x) * a.gpw : blockIdx.x / a.splits;
    const int part0 = whole ? 0 : static_cast<int>(blockIdx.x - g0 * a.splits);
    const int here = !whole ? 1 : (a.G - g0 < a.gpw ? static_cast<int>(a.G - g0) : a.gpw);

    // masks: a wave reads the rows of groups wv, wv + 4, .. (N < 64: one ballot each)
    constexpr int kMaskRows = 4;
    for (int q0 = wv; q0 < a.gpw; q0 += kMaskRows * kPairWaves) {
        uint8_t byte[kMaskRows];
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int q = q0 + u * kPairWaves;
            byte[u] = a.mask[q < here && lane < N ? (g0 + q) * N + lane : g0 * N];
        }
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int q = q0 + u * kPairWaves;
            if (q >= here) break;
            const bool b = lane < N && byte[u] != 0;
            const unsigned long long m = __ballot(b);
            const int n = static_cast<int>(__popcll(m));
            const bool good = n == N - S;
            if (lane == 0) {
                bits[q] = good ? m : 0ull;
                if ((whole || a.splits == 1) && a.status != nullptr) a.status[g0 + q] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
            }
        }
    }
    const double alpha = nodes.alpha[(lane & 15) < K ? lane & 15 : 0];
    if (tid < N) beta_s[tid] = nodes.beta[tid];
    if constexpr (HOMOG) {
        constexpr int MH = Tile::kMH;
        if (tid < 2 * MH * MH) mono[tid] = kChebyshev.c[tid / (MH * MH)][tid / MH % MH][tid % MH];
    }
    for (int e = tid; e < kWave * a.gpw; e += kPairThreads) votes[e] = 0;
    if (tid < 16) hit[tid] = -1;
    __syncthreads();
    if (!whole && bits[0] == 0ull) return;

    const unsigned long long all = (1ull << N) - 1ull;
    const double lift = h ? a.lift1 : a.lift0;
    const int slot = wv * kPairsPerWave + lane / 2;
    const int Cs = whole ? static_cast<int>(a.C) : kPairClasses;            // classes of a row of the tile
    const int C = static_cast<int>(a.C);
    const int q = whole ? slot / Cs : 0;
    const int c_rel = slot - q * Cs;                      // parts: slot < 128 = Cs
    const char *src = reinterpret_cast<const char *>(a.preds + static_cast<size_t>(g0) * N * a.C);
    for (int part = part0; MODE == kParts ? part < a.parts : part == part0; part += MODE == kParts ? a.splits : 1) {
        const int c = part * kPairClasses + c_rel;
        const bool in = q < here && c < C;
        const unsigned long long rows = in ? bits[q] : 0ull;
        const bool live = rows != 0ull;
        float *y = Ysh + (in ? q * N * Cs + c_rel : 0);
        // lane h of the pair brings the rows of workers h, h + 2, ..; both lanes then read all of them.  In place of a row
        // that is missing, and is not to be read, goes the first one that is there.
        float pf[Tile::kNodes];
        const unsigned long long own_rows = rows >> h;    // bit 2u: row of load u
        if (live) {
            const unsigned first = 4u * static_cast<unsigned>((q * N + __builtin_ctzll(rows)) * C + c);
            unsigned at = 4u * static_cast<unsigned>((q * N + h) * C + c);
#pragma unroll
            for (int u = 0; u < Tile::kNodes; ++u, at += 8u * C)
                pf[u] = *reinterpret_cast<const float *>(src + ((own_rows & (1ull << (2 * u))) != 0ull ? at : first));
        }
        if (part == part0) {                              // meanwhile the tables
            pair_table<MT, TQ, S>(tab, N, beta_s);
            if (whole) {                                  // lane = query, a worker to each row of lanes
#pragma unroll
                for (int u = 0; u < (2 * Tile::kNodes + kPairRows - 1) / kPairRows; ++u) {
                    const int i = u * kPairRows + tid / 16;
                    const double d = alpha - beta_s[i < N ? i : 0];
                    const bool at = d == 0.0;             // nodes are distinct: one worker at most
                    if (i < N) {
                        T[i * 16 + (lane & 15)] = at ? 0.0 : rcp_normal(d);
                        if (at && (lane & 15) < K) hit[lane & 15] = i;
                    }
                }
            }
        }
        if (live) {
#pragma unroll
            for (int u = 0; u < Tile::kNodes; ++u)
                if (2 * u + h < N) y[(2 * u + h) * Cs] = (own_rows & (1ull << (2 * u))) != 0ull ? pf[u] : 0.0f;
        }
        if (part == part0) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
        int Np = N, Mp = M, Ap = A, hp = h;
        // parts: nothing of what follows is worth carrying from one to the next, registers being what is short
        if (MODE == kParts) asm volatile("" : "+s"(Np), "+s"(Mp), "+s"(Ap), "+v"(hp));
        if (whole ? wv * kPairsPerWave < here * Cs : part * kPairClasses + wv * kPairsPerWave < C) {   // else: no class, the rest only
            const bool settled = locate_class_pair<MT, TQ, S, HOMOG>(y, Cs, rows, all & ~rows, tab, mono + hp * Tile::kMH * Tile::kMH, Np,
                                                                     Mp, Ap, hp, lift, live, votes + kWave * (in ? q : 0));
            if constexpr (HOMOG) {
                unsigned long long open = __ballot(live && !settled && h == 0);
                const int n = N - S, per_wave = pair_scratch_doubles(N, n, M);
                double *xs = scratch + wv * per_wave, *mat = xs + N;
                int *avail = reinterpret_cast<int *>(mat + n * (2 * M + 1) + M + n);
                while (open != 0ull) {                    // the whole wave on one class
                    const int from = __builtin_ctzll(open);
                    open &= open - 1ull;
                    const int qf = __builtin_amdgcn_readlane(in ? q : 0, from), cf = __builtin_amdgcn_readlane(c, from);
                    const unsigned long long there = bits[qf];
                    if (lane < N && ((there >> lane) & 1ull)) {
                        const int at = __popcll(there & ((1ull << lane) - 1ull));
                        avail[at] = lane;
                        xs[at] = beta_s[lane];
                    }
                    __builtin_amdgcn_wave_barrier();
                    locate_classes_wave<true>(a.preds + static_cast<size_t>(g0 + qf) * N * a.C, a.C, cf, 1, avail, xs, n, M, A, mat,
                                              votes + kWave * qf, true);
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
        __builtin_amdgcn_wave_barrier();                  // the next part's rows: this pair's own places again
    }
    __syncthreads();

    if constexpr (!whole) {
        if (MODE == kPart || a.splits > 1) {              // the words are read by the next launch
            if (tid < N && votes[tid] != 0)
                __hip_atomic_fetch_add(&a.votes[g0 * (N + 1) + tid], votes[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if constexpr (MODE == kParts) {
            const int KP = round_up4(K), nF = N - S - A;
            double *WdT = reinterpret_cast<double *>(Ysh), *alpha_s = WdT + nF * KP;      // located_lds_bytes <= the tile's N x 128 floats
            int *F = reinterpret_cast<int *>(alpha_s + K);
            const unsigned long long drop = most_voted(votes, N, A), left = bits[0] & ~drop, below = (1ull << lane) - 1ull;
            if (wv == 0 && ((drop >> lane) & 1ull)) a.adv[g0 * A + __popcll(drop & below)] = lane;
            if (wv == 0 && ((left >> lane) & 1ull)) F[__popcll(left & below)] = lane;
            if (tid < K) alpha_s[tid] = nodes.alpha[tid];
            for (int e = tid; e < nF * KP; e += kPairThreads) WdT[e] = 0.0;
            __syncthreads();
            decoder_weights(alpha_s, beta_s, F, nF, K, KP, a.sign_mode, WdT);
            __syncthreads();
            const float *pg = a.preds + static_cast<size_t>(g0) * N * a.C;
            float *og = a.out + static_cast<size_t>(g0) * K * a.C;
            if (a.vec4) contract_columns<4, (MT + 2) / 4>(pg, og, F, nF, K, KP, a.C, a.C / 4, WdT);     // K < MT
            else contract_columns<1, (MT + 2) / 4>(pg, og, F, nF, K, KP, a.C, a.C, WdT);
        }
        return;
    } else {

        // two or four rows share the workers of a unit (sixteen classes of a group) where the workgroup has that many to spare
        const int l = lane & 15;
        const int chunks = (Cs + 15) / 16, units = here * chunks;
        const int share = units * 4 <= kPairRows ? 2 : (units * 2 <= kPairRows ? 1 : 0);           // log2
        const int sub = (lane / 16) & ((1 << share) - 1), per_wave = 4 >> share;
        double *sg = sgn + (wv * 4 + lane / 16) * N;
        for (int u0 = wv * per_wave; u0 < units; u0 += kPairWaves * per_wave) {
            const int unit = u0 + ((lane / 16) >> share);
            const int q = unit < units ? unit / chunks : 0;
            const int c = (unit - q * chunks) * 16 + l;
            const unsigned long long there = bits[q];
            const bool live = unit < units && there != 0ull;
            // the A most voted workers, equal counts: smaller index first.  Every class gives A distinct workers a vote, so
            // at least A have one.
            int key[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const int w = l + 16 * p;
                key[p] = p < 2 || N > 32 ? (w < N ? (votes[q * kWave + w] << 6) | (kWave - 1 - w) : -1) : -1;
            }
            unsigned drop = 0u, drop_high = 0u;           // workers 0 .. 31, 32 ..
            int located = 0;                              // lane k < A: the k-th of the located workers, in ascending order
#pragma unroll
            for (int pick = 0; pick < kPairMaxAdversaries; ++pick) {
                if (pick >= A) break;
                int m = max(key[0], max(key[1], key[2]));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor1, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor2, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowHalfMirror, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowMirror, 0xF, 0xF, true));
                const int w = kWave - 1 - (m & (kWave - 1));
                drop |= w < 32 ? 1u << w : 0u;
                drop_high |= w < 32 ? 0u : 1u << (w - 32);
#pragma unroll
                for (int p = 0; p < 3; ++p) key[p] = key[p] == m ? -1 : key[p];          // keys of workers differ
            }
            {
                unsigned long long rest = drop | static_cast<unsigned long long>(drop_high) << 32;
#pragma unroll
                for (int k = 0; k < kPairMaxAdversaries; ++k) {
                    located = l == k ? __builtin_ctzll(rest | 1ull << 63) : located;
                    rest &= rest - 1ull;
                }
                if (live && c < A && sub == 0) a.adv[(g0 + q) * A + l] = located;         // the group's first chunk: c = l
            }
            const unsigned left = static_cast<unsigned>(there) & ~drop, left_high = static_cast<unsigned>(there >> 32) & ~drop_high;
            const auto sign = [&](int w, unsigned of, int before, int at) {              // w: bit of `of`; `before` are left ahead of it
                const int odd = a.sign_mode == APPROXIFER_SIGN_SURVIVOR_RANK ? before + __popc(of & ((1u << w) - 1u)) : w;
                sg[at] = __hiloint2double((of >> w) & 1u ? 0x3ff00000 | odd << 31 : 0, 0);                 // 1, -1 or 0
            };
            if (l < N) sign(l, left, 0, l);
            if (l + 16 < N) sign(l + 16, left, 0, l + 16);
            if (N > 32 && l + 32 < N) sign(l, left_high, __popc(left), l + 32);
            __builtin_amdgcn_wave_barrier();
            const float *y = Ysh + q * N * Cs + (c < Cs ? c : 0);
            // Four sums, over the workers 4 m + r of each r, added as (0 + 1) + (2 + 3) whichever rows of lanes have taken them: how many
            // groups lie in a workgroup is not to show in a group's bits.
            double acc[MT - 1], den;                      // K < M <= MT
            const auto contract = [&](auto rows) {        // 1, 2 or 4 rows to a unit, each with 4, 2 or 1 of the sums
                constexpr int kRows = decltype(rows)::value, kSums = 4 / kRows, kAhead = 4;
                double part[kSums][MT - 1], dens[kSums];
#pragma unroll
                for (int r = 0; r < kSums; ++r) {
                    dens[r] = 0.0;
#pragma unroll
                    for (int j = 0; j < MT - 1; ++j) part[r][j] = 0.0;
                }
                const double *sp = sg + sub, *tp = T + sub * 16 + l;
                const float *yp = y + sub * Cs;
                const int ystride = Cs * kRows;
                const auto block = [&](int room) {        // the next four workers of this row, `room` of them and more there
                    double s[kAhead], ti[kAhead];
                    float yi[kAhead];
#pragma unroll
                    for (int b = 0; b < kAhead; ++b) {
                        const int at = b < room ? b : 0;
                        s[b] = b < room ? sp[at * kRows] : 0.0;
                        ti[b] = tp[at * 16 * kRows];
                        yi[b] = yp[at * ystride];
                    }
#pragma unroll
                    for (int b = 0; b < kAhead; ++b) {
                        const double v = s[b] * static_cast<double>(s[b] != 0.0 ? yi[b] : 0.0f);   // who is out may hold anything
                        row_outer<0, 0, MT - 1>(part[b % kSums], ti[b], v);
                        dens[b % kSums] = fma(ti[b], s[b], dens[b % kSums]);
                    }
                    sp += kAhead * kRows;
                    tp += kAhead * 16 * kRows;
                    yp += kAhead * ystride;
                };
                const int full = N / (kRows * kAhead);    // blocks that every row of the unit has whole
                for (int b = 0; b < full; ++b) block(kAhead);
                for (int i = sub + full * kAhead * kRows; i - sub < N; i += kAhead * kRows) {
                    const int room = (N - i + kRows - 1) / kRows;           // none, for the last rows: 0
                    if (room <= 0) {
                        sp = sg;
                        tp = T + l;
                        yp = y;
                    }
                    block(room);
                }
                const auto total = [&](auto of) {
                    if constexpr (kRows == 1) return (of(0) + of(1)) + (of(2) + of(3));
                    else if constexpr (kRows == 2) return rows_sum<16>(of(0)) + rows_sum<16>(of(1));
                    else return rows_sum<32>(rows_sum<16>(of(0)));
                };
                den = total([&](int r) { return dens[r]; });
#pragma unroll
                for (int j = 0; j < MT - 1; ++j) acc[j] = total([&](int r) { return part[r][j]; });
            };
            if (share == 0) contract(std::integral_constant<int, 1>());
            else if (share == 1) contract(std::integral_constant<int, 2>());
            else contract(std::integral_constant<int, 4>());
            const double rden = rcp_normal(den);
            const int on = hit[l];                            // query l's own worker, if it is one's node
            const bool hits = __ballot(on >= 0) != 0ull;
            float *og = a.out + (static_cast<size_t>(g0) + q) * K * Cs + c;
            const bool mine = live && c < Cs;
    #pragma unroll
            for (int j = 0; j < MT - 1; ++j) {
                if (j < K) {
                    double v = acc[j] * row_bcast_dyn(rden, j);
                    if (hits) {
                        const int at = __builtin_amdgcn_readlane(on, j);
                        if (at >= 0 && ((at < 32 ? left >> at : left_high >> (at - 32)) & 1u) != 0u) v = static_cast<double>(y[at * Cs]);
                    }
                    if (mine && (j & ((1 << share) - 1)) == sub) og[j * Cs] = static_cast<float>(v);
                }
            }
            __builtin_amdgcn_wave_barrier();                  // before the signs of the next groups
        }
    }
}

template <int MT, int TQ, int S, bool HOMOG>
int run_pairs(const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    const bool whole = call.parts == 1;
    const size_t lds = pair_lds_bytes<MT, TQ, S>(whole, call.gpw, call.N, call.K + call.A, call.C, HOMOG);
    auto kernel = whole ? decode_byzantine_pairs_kernel<MT, TQ, S, kWhole, HOMOG> : decode_byzantine_pairs_kernel<MT, TQ, S, kParts, HOMOG>;
    if constexpr (!HOMOG) {
        if (call.splits > 1) kernel = decode_byzantine_pairs_kernel<MT, TQ, S, kPart, HOMOG>;
    }
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    const int64_t blocks = whole ? (call.G + call.gpw - 1) / call.gpw : call.G * call.splits;
    return launch_status(launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kPairThreads), lds, stream, call, nodes));
}

// M rounded up to even, TQ = MT / 2 or one more.
template <int MT, int TQ, bool HOMOG>
int run_pairs_rows(const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    switch (call.S) {
        case 0: return run_pairs<MT, TQ, 0, HOMOG>(call, nodes, stream);
        case 1: return run_pairs<MT, TQ, 1, HOMOG>(call, nodes, stream);
        case 2: return run_pairs<MT, TQ, 2, HOMOG>(call, nodes, stream);
        case 3: return run_pairs<MT, TQ, 3, HOMOG>(call, nodes, stream);
        default: return run_pairs<MT, TQ, 4, HOMOG>(call, nodes, stream);
    }
}
template <int MT, bool HOMOG>
int run_pairs_columns(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return tq == MT / 2 ? run_pairs_rows<MT, MT / 2, HOMOG>(call, nodes, stream) : run_pairs_rows<MT, MT / 2 + 1, HOMOG>(call, nodes, stream);
}
// one function per MT and locator, spread over source files for the build's sake
int run_pairs_4(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_6(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_8(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_10(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_12(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_14(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_16(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_4(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_6(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_8(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_10(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_12(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_null_pairs_14(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);

}  // namespace approxifer

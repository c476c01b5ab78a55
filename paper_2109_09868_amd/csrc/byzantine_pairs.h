// Algorithm 2 on the library's own worker nodes, beta_i = cos(i pi / (N - 1)), with at most four workers missing: two
// lanes to a class.
#pragma once

#include "byzantine_common.h"
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
    int32_t *adv, *status, *votes;
    int64_t G, C;
    int K, N, S, A, sign_mode;
    int gpw;                 // groups of a workgroup (whole groups), or
    int parts, splits;       // parts > 1: parts of a group's classes, each with a workgroup of its own (splits = parts) or one (1)
    double lift0, lift1;     // see locate_class_pair
};

// x or y by a condition, as values: the compiler otherwise turns a choice between neighbouring elements of an array into
// one element at an address of its own, and keeps the array in memory for it.
__device__ __forceinline__ double choose(bool first, double x, double y) {
    asm("" : "+v"(x), "+v"(y));
    return first ? x : y;
}
__device__ __forceinline__ double pair_other(double v) { return dpp_exchange<kDppQuadXor1>(v); }
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

// Algorithm 2, steps 1-5, for the class of this pair of lanes; h = lane % 2.
//
// The polynomial P is eliminated in closed form.  With omega = (1/2, 1, .., 1, 1/2) the Chebyshev polynomials are orthogonal
// on the nodes, so the rows u_r = omega T_{N-1-r} = w T_r, r < R = N - M, are orthogonal to every polynomial of degree
// below M; their Gram matrix in the plain inner product is diagonal but for -1/2 between rows of equal parity, a rank-one
// term for either parity, whose inverse root (1 + lift e e^T per parity, e_0 = sqrt(1/2), else 1) makes them orthonormal.
// In the same basis for Q the system's entries are sums of two moments,
//     u_r diag(y) T_e = (lambda_{r+e} + lambda_|r-e|) / 2,     lambda_t = sum_i w_i y_i T_t(beta_i),
// and the mirror images beta_{N-1-i} = -beta_i halve the work for the moments: no factorisation of the nodes, and a sixth
// of the multiply-adds of forming U diag(y) V entry by entry.  A missing worker's prediction counts as a free unknown (its
// column u_r e_i is eliminated ahead of the class's own, y_i = 0).  Q_0 = 1 is sum_e q_e T_e(0) = 1, which takes the even
// columns to T_e - T_e(0).
// Rows of parity h live in lane h (row 2t + h in slot t): the moments of a parity, the rank-one term and the even and odd
// part of Q are a lane's own, and a dot product over the rows is two short ones and an exchange.  The elimination is
// modified Gram-Schmidt on [missing | columns 1 .. M-1 | column 0], as backward stable here as Householder reflections
// with the right-hand side carried along (Bjorck 1967).  Next to the monomial basis its solutions are closer to the exact
// ones: largest error of Q(x_i) relative to their maximum over 60 draws (both forms in numpy), K = 12, A = 2, 28 workers 2e-9 and 2e-8, K = 8, A =
// 2, 20 of 24 workers 1.4e-10 and 5e-10.
//   y, ys: the class's predictions, y[i ys] for worker i (LDS), zero where there is no answer
//   bits: workers that answered, missing: the others;  votes: the group's counters;  live: the pair has a class
template <int MT, int TQ, int S>
__device__ __forceinline__ void locate_class_pair(const float *y, int ys, unsigned long long bits, unsigned long long missing,
                                                  const double *tab, int N, int M, int A, int h, double lift, bool live,
                                                  int *votes) {
    typedef PairTile<MT, TQ, S> Tile;
    typedef double v2d __attribute__((ext_vector_type(2)));
    constexpr int TT = Tile::TT, MH = Tile::kMH, kLam = Tile::kLam, kRow = 2 * Tile::kLamPad;
    const int NH = (N + 1) / 2;
    const int R = N - M;
    const double mirror = ((N - 1 + h) & 1) ? -1.0 : 1.0;  // w_{N-1-i} T_t(beta_{N-1-i}) against node i, t of parity h
    const double *own = tab + h * Tile::kLamPad;

    // ---- moments: p[s] = lambda_{2s+h}, o[s] = lambda_{2s+1-h} -----------------------------------------------------------
    double p[Tile::kLamPad];
#pragma unroll
    for (int s = 0; s < Tile::kLamPad; ++s) p[s] = 0.0;
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
            const double z = fma(mirror, static_cast<double>(hi[i & 1]), static_cast<double>(lo[i & 1]));
#pragma unroll
            for (int s = 0; s < kReads; ++s) {
                p[2 * s] = fma(row[i & 1][s][0], z, p[2 * s]);
                p[2 * s + 1] = fma(row[i & 1][s][1], z, p[2 * s + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
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
        if (u > 0) {
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

    // ---- elimination: nf[j][e / 2] = minus the share of column j in column e, lane e % 2 keeping it ------------------------
    double nf[MT][MH];
#pragma unroll
    for (int j = 1; j < MT; ++j) {
        if (j < M) {
            double sig = a[j][0] * a[j][0];
#pragma unroll
            for (int t = 1; t < TQ; ++t) sig = fma(a[j][t], a[j][t], sig);
            const double rs = rcp_normal(pair_sum(sig));
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
    double c[MH], part[MT];
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

    // ---- a_i = Q(beta_i), up to sign: lane 0 node i, lane 1 its mirror image; the A smallest vote --------------------------
    // The three smallest so far, worker in the low six bits: equal magnitudes, and what agrees to 46 bits, in worker order.
    const unsigned answered = static_cast<unsigned>(h ? __brevll(bits) >> (64 - N) : bits);
    const unsigned mine = answered & ((1u << (h ? N / 2 : NH)) - 1u);    // bit i: this lane's node i; a middle one is lane 0's
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
            v = min_magnitude(v, 1e300);                  // not a number: behind every number
            // nor does a worker that did not answer, or a row past the last node, come before any that did
            const bool there = S > 0 ? (mine & (1u << i)) != 0u : i < Tile::kNodes - 4 || (i < NH && !(h && 2 * i == N - 1));
            const double k = __hiloint2double(there ? __double2hiint(v) : 0x7fe00000,
                                              (__double2loint(v) & ~63) | (h ? N - 1 - i : i));
            l2 = min_number(l2, max_number(l1, k));
            l1 = min_number(l1, max_number(l0, k));
            l0 = min_number(l0, k);
        }
    }
    // of two ascending lists of A, the A smallest are those where own k-th < the other's (A - 1 - k)-th, from either side
    const double m0 = pair_other(l0), m1 = pair_other(l1), m2 = pair_other(l2);
    const auto vote = [&](double k, double against) {
        if (live && k < against) atomicAdd(&votes[__double2loint(k) & 63], 1);
    };
    vote(l0, A == 1 ? m0 : (A == 2 ? m1 : m2));
    if (A > 1) vote(l1, A == 2 ? m0 : m1);
    if (A > 2) vote(l2, m0);
}

// A workgroup takes `gpw` whole groups (C <= 128), a class to a pair of lanes, and decodes them, a row
// of sixteen lanes to sixteen classes of a group:
//     out[j][c] = (sum_i T[j][i] s_i y_ic) / (sum_i T[j][i] s_i),     T[j][i] = 1 / (alpha_j - beta_i),
// lane j of the row holding T[j][i], which reaches the classes inside the multiply-add and sums the denominator of query j;
// s_i is the sign of worker i, 0 if it does not count.  A query node that is a worker's node has T = 0 there and takes that
// worker's row.  More classes: a workgroup to every 128 of a group's (kPart), or one that takes them all in turn (kParts: the
// workgroups cannot meet without a workspace; the loop costs 50 registers, and with them the second wave of a SIMD); the
// last to finish writes the located workers, and decode_located_kernel decodes.  No row of a worker that did not answer is read.
// dynamic LDS: double tab | beta_s[N] | whole groups: T[N][16] | sgn[16][N]
//              | float Ysh[groups][N][classes] | uint64 bits[gpw] | int votes[gpw][64] | hit[16]
__host__ __device__ constexpr int pair_decode_doubles(bool whole, int N) {
    const int d = whole ? 16 * N + kPairRows * N + N : N;
    return (d + 1) & ~1;
}
__host__ __device__ constexpr int64_t pair_tile_floats(bool whole, int gpw, int N, int64_t C) {
    return ((whole ? gpw * N * C : static_cast<int64_t>(N) * kPairClasses) + 3) & ~static_cast<int64_t>(3);
}
template <int MT, int TQ, int S>
constexpr size_t pair_lds_bytes(bool whole, int gpw, int N, int64_t C) {
    return sizeof(double) * (PairTile<MT, TQ, S>::kTableDoubles + pair_decode_doubles(whole, N)) +
           sizeof(float) * pair_tile_floats(whole, gpw, N, C) + sizeof(uint64_t) * gpw + sizeof(int) * (kWave * gpw + 16);
}

enum PairMode { kWhole, kPart, kParts };

template <int MT, int TQ, int S, PairMode MODE>
constexpr int kPairWavesPerSimd = MT * TQ + S * (TQ + (S + 1) / 2) <= (MODE == kParts ? 60 : 100) ? 2 : 1;

template <int MT, int TQ, int S, PairMode MODE>
__global__ __launch_bounds__(kPairThreads) __attribute__((amdgpu_waves_per_eu(kPairWavesPerSimd<MT, TQ, S, MODE>))) void decode_byzantine_pairs_kernel(
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
                if (part0 == 0 && a.status != nullptr) a.status[g0 + q] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
            }
        }
    }
    const double alpha = nodes.alpha[(lane & 15) < K ? lane & 15 : 0];
    if (tid < N) beta_s[tid] = nodes.beta[tid];
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
    for (int part = part0; MODE == kParts ? part < a.parts : part == part0; ++part) {
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
        if (whole ? wv * kPairsPerWave < here * Cs : part * kPairClasses + wv * kPairsPerWave < C)   // else: no class, the rest only
            locate_class_pair<MT, TQ, S>(y, Cs, rows, all & ~rows, tab, Np, Mp, Ap, hp, lift, live, votes + kWave * (in ? q : 0));
        __builtin_amdgcn_wave_barrier();                  // the next part's rows: this pair's own places again
    }
    __syncthreads();

    if constexpr (!whole) {
        if (MODE == kPart && !pool_votes_last_arrival(a.votes + g0 * (N + 1), votes, N, a.splits, hit)) return;
        if (wv != 0) return;
        // as below, a lane to a worker
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
        if ((drop >> lane) & 1ull) a.adv[g0 * A + __popcll(drop & ((1ull << lane) - 1ull))] = lane;
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
            double acc[MT - 1], den = 0.0;                // K < M <= MT
#pragma unroll
            for (int j = 0; j < MT - 1; ++j) acc[j] = 0.0;
            const double *sp = sg + sub, *tp = T + sub * 16 + l;
            const float *yp = y + sub * Cs;
            constexpr int kAhead = 4;
            const int stride = 1 << share, ystride = Cs << share;
            const auto block = [&](int room) {            // the next four workers of this row, `room` of them and more there
                double s[kAhead], ti[kAhead];
                float yi[kAhead];
#pragma unroll
                for (int b = 0; b < kAhead; ++b) {
                    const int at = b < room ? b : 0;
                    s[b] = b < room ? sp[at * stride] : 0.0;
                    ti[b] = tp[at * 16 * stride];
                    yi[b] = yp[at * ystride];
                }
#pragma unroll
                for (int b = 0; b < kAhead; ++b) {
                    const double v = s[b] * static_cast<double>(s[b] != 0.0 ? yi[b] : 0.0f);   // who is out may hold anything
                    row_outer<0, 0, MT - 1>(acc, ti[b], v);
                    den = fma(ti[b], s[b], den);
                }
                sp += kAhead * stride;
                tp += kAhead * 16 * stride;
                yp += kAhead * ystride;
            };
            const int full = (N >> share) / kAhead;       // blocks that every row of the unit has whole
            for (int b = 0; b < full; ++b) block(kAhead);
            for (int i = sub + full * kAhead * stride; i - sub < N; i += kAhead * stride) {
                const int room = (N - i + stride - 1) >> share;          // none, for the last rows: 0
                if (room <= 0) {
                    sp = sg;
                    tp = T + l;
                    yp = y;
                }
                block(room);
            }
            if (share > 0) {
                den = rows_sum<16>(den);
#pragma unroll
                for (int j = 0; j < MT - 1; ++j) acc[j] = rows_sum<16>(acc[j]);
            }
            if (share > 1) {
                den = rows_sum<32>(den);
#pragma unroll
                for (int j = 0; j < MT - 1; ++j) acc[j] = rows_sum<32>(acc[j]);
            }
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

template <int MT, int TQ, int S>
int run_pairs(const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    const bool whole = call.parts == 1;
    const size_t lds = pair_lds_bytes<MT, TQ, S>(whole, call.gpw, call.N, call.C);
    const auto kernel = whole ? decode_byzantine_pairs_kernel<MT, TQ, S, kWhole>
                              : (call.splits > 1 ? decode_byzantine_pairs_kernel<MT, TQ, S, kPart>
                                                 : decode_byzantine_pairs_kernel<MT, TQ, S, kParts>);
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    const int64_t blocks = whole ? (call.G + call.gpw - 1) / call.gpw : call.G * call.splits;
    return launch_status(launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kPairThreads), lds, stream, call, nodes));
}

// M rounded up to even, TQ = MT / 2 or one more.
template <int MT, int TQ>
int run_pairs_rows(const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    switch (call.S) {
        case 0: return run_pairs<MT, TQ, 0>(call, nodes, stream);
        case 1: return run_pairs<MT, TQ, 1>(call, nodes, stream);
        case 2: return run_pairs<MT, TQ, 2>(call, nodes, stream);
        case 3: return run_pairs<MT, TQ, 3>(call, nodes, stream);
        default: return run_pairs<MT, TQ, 4>(call, nodes, stream);
    }
}
template <int MT>
int run_pairs_columns(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream) {
    return tq == MT / 2 ? run_pairs_rows<MT, MT / 2>(call, nodes, stream) : run_pairs_rows<MT, MT / 2 + 1>(call, nodes, stream);
}
// one function per MT, spread over source files for the build's sake
int run_pairs_4(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_6(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_8(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_10(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_12(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_14(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);
int run_pairs_16(int tq, const PairCall &call, const Nodes &nodes, hipStream_t stream);

}  // namespace approxifer

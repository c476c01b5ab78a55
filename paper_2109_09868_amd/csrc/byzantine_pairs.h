// Algorithm 2 on the library's own worker nodes, beta_i = cos(i pi / (N - 1)), with at most four workers missing: two
// lanes to a class.
#pragma once

#include "byzantine_common.h"
#include "rows.h"

namespace approxifer {

constexpr int kPairsPerWave = kWave / 2;
constexpr int kPairMaxAdversaries = 3;
constexpr int kPairMaxMissing = 4;
constexpr int kPairMaxWaves = 4;
constexpr int kPairPart = kPairMaxWaves * kPairsPerWave;   // classes of a workgroup that has part of a group's

// Launch arguments of decode_byzantine_pairs_kernel, by value.
struct PairCall {
    const float *preds;
    const uint8_t *mask;
    float *out;
    int32_t *adv, *status, *votes;
    int64_t G, C, Cv;
    int K, N, S, A, n_cap, vec4, sign_mode;
    int gpw;                 // groups of a workgroup (whole groups), or
    int parts, splits;       // parts > 1: parts of a group's classes, dealt to `splits` workgroups
    double lift0, lift1;     // see locate_class_pair
};

// x or y by a condition, as values: the compiler otherwise turns a choice between neighbouring elements of an array into
// one element at an address of its own, and keeps the array in memory for it.
__device__ __forceinline__ double choose(bool first, double x, double y) {
    asm("" : "+v"(x), "+v"(y));
    return first ? x : y;
}
__device__ __forceinline__ double pair_other(double v) { return dpp_exchange<kDppQuadXor1>(v); }
__device__ __forceinline__ double rows_other(double v, int distance) {     // of lane ^ distance, 16 or 32
    return __shfl_xor(v, distance);
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

// Tile: MT >= M columns (even), TT row slots to a lane, up to SX missing workers; 2 TT >= N - M.
template <int MT, int TT>
struct PairTile {
    static constexpr int kMH = MT / 2;
    static constexpr int kLam = kMH + TT;                  // moments of one parity that the system is formed from
    static constexpr int kLamPad = (kLam + 1) & ~1;
    static constexpr int kNodes = (MT + 2 * TT + 1) / 2;   // most nodes that are not mirror images of others
    static constexpr int kTableDoubles = kNodes * 2 * kLamPad;
};

// The table tab[i][h][s] = w_i T_{2s+h}(beta_i) over the nodes i < ceil(N / 2), w_i = (-1)^i, halved at the end node and at
// a node in the middle (its own mirror image, which is counted twice); zero for i up to kNodes.  T_t(cos x) = cos t x: the
// values are nodes again.  A row of sixteen lanes takes every (rows)-th t of sixteen nodes; `beta`: LDS.
template <int MT, int TT>
__device__ __forceinline__ void pair_table(double *tab, int N, const double *beta) {
    typedef PairTile<MT, TT> Tile;
    constexpr int kTs = 2 * Tile::kLamPad, kSteps = (kTs + 3) / 4;
    const int NH = (N + 1) / 2, period = 2 * (N - 1);
    const int rows = blockDim.x / 16, r = threadIdx.x / 16;              // 4 to 16
#pragma unroll
    for (int i0 = 0; i0 < Tile::kNodes; i0 += 16) {
        const int i = i0 + threadIdx.x % 16;
        const bool node = i < NH;
        const double w = !node ? 0.0 : (i & 1 ? -1.0 : 1.0) * (i == 0 ? 0.5 : 1.0) * (2 * i == N - 1 ? 0.5 : 1.0);
        int step = node ? i * rows : 0, k = node ? i * r : 0;            // modulo the period: i * 16 <= 4 periods
#pragma unroll
        for (int m = 4; m > 0; m /= 2) {
            step = step >= m * period ? step - m * period : step;
            k = k >= m * period ? k - m * period : k;
        }
        const auto entries = [&](int u0, int u1) {
#pragma unroll
            for (int u = u0; u < u1; ++u) {
                const int t = r + u * rows;
                const double v = beta[k < N ? k : period - k];
                if (i < Tile::kNodes && t < kTs) tab[i * kTs + (t & 1) * Tile::kLamPad + t / 2] = w * v;
                k += step;
                k = k >= period ? k - period : k;
            }
        };
        entries(0, 2);                                    // four waves need no more of these, or three
        if (2 * rows < kTs) entries(2, kSteps);
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
// ones: largest error of Q(x_i) relative to their maximum over 60 draws, K = 12, A = 2, 28 workers 2e-9 and 2e-8, K = 8, A =
// 2, 20 of 24 workers 1.4e-10 and 5e-10.
//   y, ys: the class's predictions, y[i ys] for worker i (LDS), zero where there is no answer
//   bits: workers that answered, missing: the others;  votes: the group's counters;  live: the pair has a class
template <int MT, int TT, int SX>
__device__ __forceinline__ void locate_class_pair(const float *y, int ys, unsigned long long bits, unsigned long long missing,
                                                  const double *tab, int N, int M, int A, double lift, bool live, int *votes) {
    typedef PairTile<MT, TT> Tile;
    typedef double v2d __attribute__((ext_vector_type(2)));
    constexpr int MH = Tile::kMH, kLam = Tile::kLam, kRow = 2 * Tile::kLamPad;
    const int h = lane_id() & 1;
    const int NH = (N + 1) / 2;
    const int R = N - M;
    const double mirror = ((N - 1 + h) & 1) ? -1.0 : 1.0;  // w_{N-1-i} T_t(beta_{N-1-i}) against node i, t of parity h
    const double *own = tab + h * Tile::kLamPad;

    // ---- moments: p[s] = lambda_{2s+h}, o[s] = lambda_{2s+1-h} -----------------------------------------------------------
    double p[Tile::kLamPad];
#pragma unroll
    for (int s = 0; s < Tile::kLamPad; ++s) p[s] = 0.0;
    {
        const float *lo = y, *hi = y + (N - 1) * ys;
#pragma unroll
        for (int i = 0; i < Tile::kNodes; ++i, lo += ys, hi -= ys) {     // N >= kNodes; rows past NH of the table are zero
            const double z = fma(mirror, static_cast<double>(*hi), static_cast<double>(*lo));
#pragma unroll
            for (int s = 0; s < Tile::kLamPad; s += 2) {
                const v2d t = *reinterpret_cast<const v2d *>(own + i * kRow + s);
                p[s] = fma(t[0], z, p[s]);
                p[s + 1] = fma(t[1], z, p[s + 1]);
            }
        }
    }
    double o[kLam], below[MH], ahead[kLam - 1];
#pragma unroll
    for (int s = 0; s < kLam; ++s) o[s] = pair_other(p[s]);
#pragma unroll
    for (int d = 1; d < MH; ++d) below[d] = choose(h, p[d - 1], p[d]);       // lambda_{|h - 2d|}
#pragma unroll
    for (int s = 0; s < kLam - 1; ++s) ahead[s] = choose(h, o[s + 1], o[s]); // lambda_{2s+1+h}

    // ---- the system: a[e][t] = entry (2t + h, e), orthonormal rows --------------------------------------------------------
    const double first = h ? 1.0 : 0.70710678118654752440;              // sqrt(1/2) for row 0
    double a[MT][TT], x[SX > 0 ? SX : 1][TT];
    const double there0 = 2 * (TT - 2) + h < R ? 1.0 : 0.0, there1 = 2 * (TT - 1) + h < R ? 1.0 : 0.0;   // of the last rows
    const auto finish_column = [&](double (&c)[TT]) {
        c[0] *= first;
        c[TT - 2] *= there0;
        c[TT - 1] *= there1;
        double sum = first * c[0];
#pragma unroll
        for (int t = 1; t < TT; ++t) sum += c[t];
        sum *= lift;
        c[0] = fma(TT == 2 ? first * there0 : first, sum, c[0]);
#pragma unroll
        for (int t = 1; t < TT; ++t) c[t] = t < TT - 2 ? c[t] + sum : fma(t == TT - 2 ? there0 : there1, sum, c[t]);
    };
    // odd columns first: the other lane's moments are then done with
#pragma unroll
    for (int u = 0; u < MH; ++u) {
#pragma unroll
        for (int t = 0; t < TT; ++t) a[2 * u + 1][t] = ahead[t + u] + (t > u ? ahead[t > u ? t - u - 1 : 0] : o[t > u ? 0 : u - t]);
        finish_column(a[2 * u + 1]);
    }
#pragma unroll
    for (int u = 0; u < MH; ++u) {
#pragma unroll
        for (int t = 0; t < TT; ++t) a[2 * u][t] = p[t + u] + (t >= u ? p[t >= u ? t - u : 0] : below[t >= u ? 1 : u - t]);
        finish_column(a[2 * u]);
        if (u > 0) {
#pragma unroll
            for (int t = 0; t < TT; ++t) a[2 * u][t] += u % 2 ? a[0][t] : -a[0][t];      // T_{2u}(0) = (-1)^u
        }
    }

    // ---- missing workers out of every column ------------------------------------------------------------------------------
    if constexpr (SX > 0) {
#pragma unroll
        for (int s = 0; s < SX; ++s) {
            const bool there = missing != 0ull;
            const int w = there ? __builtin_ctzll(missing) : 0;
            missing &= missing - 1ull;
            const double sign = there ? (2 * w >= N ? mirror : 1.0) : 0.0;
            const double *row = own + (2 * w >= N ? N - 1 - w : w) * kRow;
#pragma unroll
            for (int t = 0; t < TT; ++t) x[s][t] = sign * row[t];
            finish_column(x[s]);
        }
#pragma unroll
        for (int s = 0; s < SX; ++s) {
            double sig = x[s][0] * x[s][0];
#pragma unroll
            for (int t = 1; t < TT; ++t) sig = fma(x[s][t], x[s][t], sig);
            sig = pair_sum(sig);
            const double rs = sig > 0.0 ? rcp_normal(sig) : 0.0;         // fewer are missing: nothing to take out
            const auto take_out = [&](double (&c)[TT]) {
                double d = x[s][0] * c[0];
#pragma unroll
                for (int t = 1; t < TT; ++t) d = fma(x[s][t], c[t], d);
                const double f = -pair_sum(d) * rs;
#pragma unroll
                for (int t = 0; t < TT; ++t) c[t] = fma(f, x[s][t], c[t]);
            };
#pragma unroll
            for (int r = s + 1; r < SX; ++r) take_out(x[r]);
#pragma unroll
            for (int e = 0; e < MT; ++e) take_out(a[e]);
        }
    }

    // ---- elimination: nf[j][e / 2] = minus the share of column j in column e, lane e % 2 keeping it ------------------------
    double nf[MT][MH];
#pragma unroll
    for (int j = 1; j < MT; ++j) {
        if (j < M) {
            double sig = a[j][0] * a[j][0];
#pragma unroll
            for (int t = 1; t < TT; ++t) sig = fma(a[j][t], a[j][t], sig);
            const double rs = rcp_normal(pair_sum(sig));
            const auto take_out = [&](double (&c)[TT]) {
                double d = a[j][0] * c[0];
#pragma unroll
                for (int t = 1; t < TT; ++t) d = fma(a[j][t], c[t], d);
                const double f = -pair_sum(d) * rs;
                if (j + 1 < MT) {                         // the right-hand side's remainder is not needed at the end
#pragma unroll
                    for (int t = 0; t < TT; ++t) c[t] = fma(f, a[j][t], c[t]);
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
#pragma unroll
        for (int i = 0; i < Tile::kNodes; ++i) {
            double v = own[i * kRow] * c[0];
#pragma unroll
            for (int s = 1; s < MH; ++s) v = fma(own[i * kRow + s], c[s], v);
            v = fma(side, pair_other(v), v);
            if (i == 0) v += v;                           // the table has half of these
            if (i >= Tile::kNodes - 4 && 2 * i == N - 1) v += v;
            v = min_magnitude(v, 1e300);                  // not a number: behind every number
            // nor does a worker that did not answer, or a row past the last node, come before any that did
            const bool there = SX > 0 ? (mine & (1u << i)) != 0u : i < Tile::kNodes - 4 || (i < NH && !(h && 2 * i == N - 1));
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

// A workgroup of up to four waves takes `gpw` whole groups (C <= 128), a class to a pair of lanes, and decodes them, a row
// of sixteen lanes to sixteen classes of a group:
//     out[j][c] = (sum_i T[j][i] s_i y_ic) / (sum_i T[j][i] s_i),     T[j][i] = 1 / (alpha_j - beta_i),
// lane j of the row holding T[j][i], which reaches the classes inside the multiply-add and sums the denominator of query j;
// s_i is the sign of worker i, 0 if it does not count.  A query node that is a worker's node has T = 0 there and takes that
// worker's row.  More classes: `splits` workgroups take turns at 128 of them each, the last to finish decodes the group.
// No row of a worker that did not answer is read.
// dynamic LDS: double tab | whole groups: T[N][16] | sgn[4 nw][N] | beta_s[N]; parts: WdT[(n_cap - A) KP] | alpha_s[K] | beta_s[N]
//              | float Ysh[groups][N][classes] | uint64 bits[gpw] | int votes[gpw][64] | hit[16]
//              | parts: avail[N] | F[N] | Fpos[N] | flag
__host__ __device__ constexpr int pair_decode_doubles(bool whole, int nw, int K, int N, int n_cap, int A) {
    const int d = whole ? 16 * N + 4 * nw * N + N : (n_cap - A) * ((K + 3) & ~3) + K + N;
    return (d + 1) & ~1;
}
__host__ __device__ constexpr int64_t pair_tile_floats(bool whole, int gpw, int N, int64_t C) {
    return ((whole ? gpw * N * C : static_cast<int64_t>(N) * kPairPart) + 3) & ~static_cast<int64_t>(3);
}
template <int MT, int TT>
constexpr size_t pair_lds_bytes(bool whole, int gpw, int nw, int K, int N, int n_cap, int A, int64_t C) {
    return sizeof(double) * (PairTile<MT, TT>::kTableDoubles + pair_decode_doubles(whole, nw, K, N, n_cap, A)) +
           sizeof(float) * pair_tile_floats(whole, gpw, N, C) + sizeof(uint64_t) * gpw +
           sizeof(int) * (kWave * gpw + 16 + (whole ? 0 : 3 * N + 2));
}

template <int MT, int TT, int SX, bool WHOLE>
__global__ __launch_bounds__(kPairMaxWaves *kWave) __attribute__((amdgpu_waves_per_eu(MT * TT <= (WHOLE ? 100 : 50) ? 2 : 1))) void decode_byzantine_pairs_kernel(
    const PairCall a, const Nodes nodes) {
    typedef PairTile<MT, TT> Tile;
    extern __shared__ __align__(16) double lds_d[];
    constexpr bool whole = WHOLE;
    const int K = a.K, N = a.N, A = a.A, M = K + A;
    const int nw = blockDim.x / kWave;
    const int tid = threadIdx.x, wv = wave_id(), lane = lane_id(), h = lane & 1;
    double *tab = lds_d;
    double *T = tab + Tile::kTableDoubles;
    double *sgn = T + 16 * N;
    double *WdT = T, *alpha_s = WdT + (a.n_cap - A) * round_up4(K);
    double *beta_s = whole ? sgn + 4 * nw * N : alpha_s + K;
    float *Ysh = reinterpret_cast<float *>(T + pair_decode_doubles(whole, nw, K, N, a.n_cap, A));
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(Ysh + pair_tile_floats(whole, a.gpw, N, a.C));
    int *votes = reinterpret_cast<int *>(bits + a.gpw);
    int *hit = votes + kWave * a.gpw;
    int *avail = hit + 16, *F = avail + N, *Fpos = F + N, *flag = Fpos + N;

    const int64_t g0 = whole ? static_cast<int64_t>(blockIdx.x) * a.gpw : blockIdx.x / a.splits;
    const int part0 = whole ? 0 : static_cast<int>(blockIdx.x - g0 * a.splits);
    const int here = !whole ? 1 : (a.G - g0 < a.gpw ? static_cast<int>(a.G - g0) : a.gpw);

    // masks: a wave reads the rows of groups wv, wv + nw, .. (N < 64: one ballot each)
    constexpr int kMaskRows = 4;
    for (int q0 = wv; q0 < a.gpw; q0 += kMaskRows * nw) {
        uint8_t byte[kMaskRows];
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int q = q0 + u * nw;
            byte[u] = a.mask[q < here && lane < N ? (g0 + q) * N + lane : g0 * N];
        }
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int q = q0 + u * nw;
            if (q >= here) break;
            const bool b = lane < N && byte[u] != 0;
            const unsigned long long m = __ballot(b);
            const int n = static_cast<int>(__popcll(m));
            const bool good = a.S < 0 ? (n >= 2 * M && n <= a.n_cap) : n == a.n_cap;
            if (lane == 0) {
                bits[q] = good ? m : 0ull;
                if (part0 == 0 && a.status != nullptr) a.status[g0 + q] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
            }
            if (!whole && b && good) avail[__popcll(m & ((1ull << lane) - 1ull))] = lane;
        }
    }
    const double alpha = nodes.alpha[(lane & 15) < K ? lane & 15 : 0];
    if (whole) {
        if (tid < N) beta_s[tid] = nodes.beta[tid];
    } else {
        stage_nodes(nodes, K, N, alpha_s, beta_s);
        for (int e = tid; e < (a.n_cap - A) * round_up4(K); e += blockDim.x) WdT[e] = 0.0;
    }
    for (int e = tid; e < kWave * a.gpw; e += blockDim.x) votes[e] = 0;
    if (tid < 16) hit[tid] = -1;
    __syncthreads();
    if (!whole && bits[0] == 0ull) return;

    const unsigned long long all = (1ull << N) - 1ull;
    const double lift = h ? a.lift1 : a.lift0;
    const int slot = wv * kPairsPerWave + lane / 2;
    const int Cs = whole ? static_cast<int>(a.C) : kPairPart;            // classes of a row of the tile
    const int C = static_cast<int>(a.C);
    const int q = whole ? slot / Cs : 0;
    const int c_rel = slot - q * Cs;                      // parts: slot < 128 = Cs
    const char *src = reinterpret_cast<const char *>(a.preds + static_cast<size_t>(g0) * N * a.C);
    for (int part = part0; part < (whole ? 1 : a.parts); part += whole ? 1 : a.splits) {
        const int c = part * kPairPart + c_rel;
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
            pair_table<MT, TT>(tab, N, beta_s);
            if (whole) {                                  // lane = query, a worker to each row of lanes
                const int rows = blockDim.x / 16;
                const auto workers = [&](int u0, int u1) {
#pragma unroll
                    for (int u = u0; u < u1; ++u) {
                        const int i = u * rows + tid / 16;
                        const double d = alpha - beta_s[i < N ? i : 0];
                        const bool at = d == 0.0;         // nodes are distinct: one worker at most
                        if (i < N) {
                            T[i * 16 + (lane & 15)] = at ? 0.0 : rcp_normal(d);
                            if (at && (lane & 15) < K) hit[lane & 15] = i;
                        }
                    }
                };
                workers(0, 3);
                if (3 * rows < N) workers(3, (Tile::kNodes + 1) / 2);
            }
        }
        if (live) {
#pragma unroll
            for (int u = 0; u < Tile::kNodes; ++u)
                if (2 * u + h < N) y[(2 * u + h) * Cs] = (own_rows & (1ull << (2 * u))) != 0ull ? pf[u] : 0.0f;
        }
        if (part == part0) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
        locate_class_pair<MT, TT, SX>(y, Cs, rows, all & ~rows, tab, N, M, A, lift, live, votes + kWave * (in ? q : 0));
        __builtin_amdgcn_wave_barrier();                  // the next part's rows: this pair's own places again
    }
    __syncthreads();

    if constexpr (!whole) {
        float *og = a.out + static_cast<size_t>(g0) * K * a.C;
        if (a.splits > 1 && !pool_votes_last_arrival(a.votes + g0 * (N + 1), votes, N, a.splits, flag)) return;
        finish_group(a.preds + static_cast<size_t>(g0) * N * a.C, og, a.adv + g0 * A, avail,
                     static_cast<int>(__popcll(bits[0])), N, A, K, round_up4(K), a.C, a.Cv, a.vec4 != 0, a.sign_mode, alpha_s,
                     beta_s, votes, F, Fpos, WdT);
        return;
    } else {

        // two or four rows share the workers of a unit (sixteen classes of a group) where the workgroup has that many to spare
        const int l = lane & 15;
        const int chunks = (Cs + 15) / 16, units = here * chunks;
        const int share = units * 4 <= nw * 4 ? 2 : (units * 2 <= nw * 4 ? 1 : 0);           // log2
        const int sub = (lane / 16) & ((1 << share) - 1), per_wave = 4 >> share;
        double *sg = sgn + (wv * 4 + lane / 16) * N;
        for (int u0 = wv * per_wave; u0 < units; u0 += nw * per_wave) {
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
            unsigned long long drop = 0ull;
#pragma unroll
            for (int pick = 0; pick < kPairMaxAdversaries; ++pick) {
                if (pick >= A) break;
                int m = max(key[0], max(key[1], key[2]));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor1, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppQuadXor2, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowHalfMirror, 0xF, 0xF, true));
                m = max(m, __builtin_amdgcn_update_dpp(0, m, kDppRowMirror, 0xF, 0xF, true));
                drop |= 1ull << (kWave - 1 - (m & (kWave - 1)));
#pragma unroll
                for (int p = 0; p < 3; ++p) key[p] = key[p] == m ? -1 : key[p];          // keys of workers differ
            }
            const unsigned long long left = there & ~drop;
            const auto sign = [&](int w) {
                const unsigned long long before = (1ull << w) - 1ull;
                const int odd = a.sign_mode == APPROXIFER_SIGN_SURVIVOR_RANK ? static_cast<int>(__popcll(left & before)) : w;
                sg[w] = __hiloint2double((left >> w) & 1ull ? 0x3ff00000 | odd << 31 : 0, 0);              // 1, -1 or 0
                if (live && c == l && sub == 0 && ((drop >> w) & 1ull)) a.adv[(g0 + q) * A + __popcll(drop & before)] = w;
            };
            if (l < N) sign(l);
            if (l + 16 < N) sign(l + 16);
            if (N > 32 && l + 32 < N) sign(l + 32);
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
            for (int d = 16; d < 16 << share; d *= 2) {
                den += rows_other(den, d);
#pragma unroll
                for (int j = 0; j < MT - 1; ++j) acc[j] += rows_other(acc[j], d);
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
                        if (at >= 0 && ((left >> at) & 1ull) != 0ull) v = static_cast<double>(y[at * Cs]);
                    }
                    if (mine && (j & ((1 << share) - 1)) == sub) og[j * Cs] = static_cast<float>(v);
                }
            }
            __builtin_amdgcn_wave_barrier();                  // before the signs of the next groups
        }
    }
}

template <int MT, int TT, int SX>
int run_pairs(PairCall call, int nw, const Nodes &nodes, hipStream_t stream) {
    const bool whole = call.parts == 1;
    const size_t lds = pair_lds_bytes<MT, TT>(whole, call.gpw, nw, call.K, call.N, call.n_cap, call.A, call.C);
    const auto kernel = whole ? decode_byzantine_pairs_kernel<MT, TT, SX, true> : decode_byzantine_pairs_kernel<MT, TT, SX, false>;
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    const int64_t blocks = whole ? (call.G + call.gpw - 1) / call.gpw : call.G * call.splits;
    return launch_status(launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(nw * kWave), lds, stream, call, nodes));
}

// One function per M (rounded up to even), each in a source file of its own choosing: extra = TT - MT / 2 - SX / 2.
template <int MT>
int run_pairs_columns(int missing, int extra, const PairCall &call, int nw, const Nodes &nodes, hipStream_t stream) {
    if (missing == 0) return extra ? run_pairs<MT, MT / 2 + 1, 0>(call, nw, nodes, stream) : run_pairs<MT, MT / 2, 0>(call, nw, nodes, stream);
    if (missing <= 2) return extra ? run_pairs<MT, MT / 2 + 2, 2>(call, nw, nodes, stream) : run_pairs<MT, MT / 2 + 1, 2>(call, nw, nodes, stream);
    return extra ? run_pairs<MT, MT / 2 + 3, 4>(call, nw, nodes, stream) : run_pairs<MT, MT / 2 + 2, 4>(call, nw, nodes, stream);
}
int run_pairs_4(int, int, const PairCall &, int, const Nodes &, hipStream_t);
int run_pairs_6(int, int, const PairCall &, int, const Nodes &, hipStream_t);
int run_pairs_8(int, int, const PairCall &, int, const Nodes &, hipStream_t);
int run_pairs_10(int, int, const PairCall &, int, const Nodes &, hipStream_t);
int run_pairs_12(int, int, const PairCall &, int, const Nodes &, hipStream_t);
int run_pairs_14(int, int, const PairCall &, int, const Nodes &, hipStream_t);

}  // namespace approxifer

// ApproxIFER decoder and fused decoder + top-1 for gfx950 (Section 3, "ApproxIFER Decoding").
//
// The group's mask is turned into the ascending survivor list F with wavefront ballots; rows of
// missing workers are never read.  Two forms of the contraction, float64 in both:
//  * weights: the K x |F| matrix of basis functions is evaluated (a group of lanes per query node,
//    the denominator by a wavefront reduction), kept transposed in LDS and broadcast from there.
//    A workgroup per (group, tile of prediction columns), or per group for the class decision.
//  * node table: T[i][j] = 1 / (alpha_j - beta_i), the same for all groups, is evaluated once per
//    workgroup; numerators and denominators are summed over F and divided at the end.  A 16-lane
//    row per group (up to sixteen classes) or per (group, 64 classes).
#include <algorithm>

#include "decode_common.h"
#include "rows.h"
#include "sectors.h"
#include "survivors.h"

namespace approxifer {
namespace {

constexpr int kRowLanes = 16;

// ------------------------------------------------------------------------------------
// decoder kernel
// ------------------------------------------------------------------------------------
// dynamic LDS: double WdT[(N-S) * KP] | double alpha_s[K] | double beta_s[N] | int F[N] | int n
template <int VEC>
__global__ void decode_kernel(const float *__restrict__ preds, const uint8_t *__restrict__ mask,
                              float *__restrict__ out, int32_t *__restrict__ status, int K, int N, int S,
                              int64_t C, int64_t Cv, int64_t ctiles, int sign_mode, const Nodes nodes) {
    extern __shared__ double lds_d[];
    const int KP = round_up4(K);
    const int nF_cap = S < 0 ? N : N - S;          // S < 0: every group brings its own straggler count
    double *WdT = lds_d;
    double *alpha_s = WdT + nF_cap * KP;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = F + N;

    const int64_t g = blockIdx.x / ctiles;
    const int64_t ct = blockIdx.x - g * ctiles;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < nF_cap * KP; e += blockDim.x) WdT[e] = 0.0;
    if (wave_id() == 0) {
        const int n = survivors_from_mask(mask + g * N, N, F);
        if (lane_id() == 0) *n_sh = n;
    }
    __syncthreads();
    const int nF = *n_sh;
    const bool good = S < 0 ? nF >= 1 : nF == nF_cap;
    if (ct == 0 && threadIdx.x == 0 && status != nullptr)
        status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    // first chunk of this lane's prediction rows: issued now, consumed after the weights exist
    const int64_t cv0 = ct * kColsPerTile;
    const int64_t cv1 = (cv0 + kColsPerTile < Cv) ? cv0 + kColsPerTile : Cv;
    const float *pg = preds + static_cast<size_t>(g) * N * C;
    typename PredVec<VEC>::type first[kRowChunk];
    {
        const int64_t cv = cv0 + (threadIdx.x % kColsPerTile);
        load_row_chunk<VEC>(pg, F, nF, 0, C, cv < cv1 ? cv : cv0, first);
    }

    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();

    contract_tile<VEC, true>(pg, out + static_cast<size_t>(g) * K * C, F, nF, K, KP, C, cv0, cv1, WdT, first);
}

// ------------------------------------------------------------------------------------
// decoder kernel with all K accumulator rows in one wave (K <= 16, 16-byte rows)
// ------------------------------------------------------------------------------------
// decode_kernel gives every quad of queries a wave of its own, so each wave moves only a third or a quarter of a
// tile's bytes, and with the registers it needs four waves fit a SIMD, which bounds the bytes in flight.  Here ONE wave
// keeps the accumulators of all K <= 4 KQ queries for its 64 vector columns, as the encoder keeps its K inputs: it
// reads every surviving row once and writes all K output rows, three to four times the bytes in flight per wave, and
// a group's tile costs one wave's worth of prologue instead of K/4.  16-byte-aligned rows, K <= 16, up to 64
// survivors; measured against decode_kernel: 512 x 12 x 1000 classes 23.1 -> 20.7 us, 4096 x 8 x 100 classes
// 17.3 -> 13.8 us, 1.1 GB (K = 16, 4096 classes) 336 -> 235 us.
// UNAL: rows are only 4-byte aligned (C % 4 != 0 or offset tensors): the same 128-bit accesses through a
// 4-byte-aligned vector type, and the lane that holds a row's last, partial vector (C % 4 floats) moves it float
// by float.  Cv = ceil(C / 4) then counts that partial vector.
// dynamic LDS: as decode_kernel.
typedef v4f v4f_dword_aligned __attribute__((aligned(4)));

template <bool UNAL>
__device__ __forceinline__ v4f load_pred_vector(const float *p, int floats) {
    // every prediction is read once and every output written once: non-temporal accesses keep them out of the way of
    // the caches (measured on the streaming kernel: 49 MB cold 21.4 -> 17.5 us, 0.4 GB 105 -> 73 us, 1.1 GB +7..9 %)
    if (!UNAL) return __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
    if (floats >= 4) return __builtin_nontemporal_load(reinterpret_cast<const v4f_dword_aligned *>(p));
    v4f v = v4f(0.0f);
    v[0] = p[0];
    if (floats > 1) v[1] = p[1];
    if (floats > 2) v[2] = p[2];
    return v;
}

template <int KQ, bool UNAL>
__global__ __launch_bounds__(kWave) void decode_stream_kernel(const float *__restrict__ preds,
                                                              const uint8_t *__restrict__ mask, float *__restrict__ out,
                                                              int32_t *__restrict__ status, int K, int N, int S, int64_t C,
                                                              int64_t Cv, int64_t ctiles, int sign_mode, const Nodes nodes) {
    constexpr int KP = 4 * KQ;
    extern __shared__ double lds_d[];
    const int nF_cap = S < 0 ? N : N - S;
    double *WdT = lds_d;
    double *alpha_s = WdT + nF_cap * KP;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);

    const int64_t g = blockIdx.x / ctiles;
    const int64_t ct = blockIdx.x - g * ctiles;
    const int lane = threadIdx.x;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = lane; e < nF_cap * KP; e += kWave) WdT[e] = 0.0;
    const int nF = survivors_from_mask(mask + g * N, N, F);
    __syncthreads();
    const bool good = S < 0 ? nF >= 1 : nF == nF_cap;
    if (ct == 0 && lane == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    const int64_t cv_raw = ct * kColsPerTile + lane;
    const bool ok = cv_raw < Cv;
    const int64_t cv = ok ? cv_raw : ct * kColsPerTile;    // lanes past the ragged end read the tile's first column
    const int floats = (UNAL && C - 4 * cv < 4) ? static_cast<int>(C - 4 * cv) : 4;   // of this lane's vector
    const float *pg = preds + static_cast<size_t>(g) * N * C + 4 * cv;
    v4f y[kRowChunk];
#pragma unroll
    for (int u = 0; u < kRowChunk; ++u)                    // in flight while the weights are evaluated
        y[u] = load_pred_vector<UNAL>(pg + static_cast<size_t>(F[u < nF ? u : nF - 1]) * C, floats);

    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();

    double acc[KP][4];
#pragma unroll
    for (int j = 0; j < KP; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.0;
    for (int r0 = 0; r0 < nF; r0 += kRowChunk) {
        if (r0 > 0) {
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u)
                y[u] = load_pred_vector<UNAL>(pg + static_cast<size_t>(F[r0 + u < nF ? r0 + u : nF - 1]) * C, floats);
        }
#pragma unroll
        for (int u = 0; u < kRowChunk; ++u) {
            if (r0 + u < nF) {
                const double *w = WdT + (r0 + u) * KP;
                const double y0 = y[u][0], y1 = y[u][1], y2 = y[u][2], y3 = y[u][3];
#pragma unroll
                for (int j = 0; j < KP; ++j) {
                    const double wj = w[j];
                    acc[j][0] = fma(wj, y0, acc[j][0]);
                    acc[j][1] = fma(wj, y1, acc[j][1]);
                    acc[j][2] = fma(wj, y2, acc[j][2]);
                    acc[j][3] = fma(wj, y3, acc[j][3]);
                }
            }
        }
    }
    if (!ok) return;
    float *og = out + static_cast<size_t>(g) * K * C + cv * 4;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        if (j < K) {
            float *dst = og + static_cast<size_t>(j) * C;
            if (!UNAL) {
                store_row<4>(dst, acc[j]);
            } else if (floats >= 4) {
                v4f v;
                v[0] = static_cast<float>(acc[j][0]);
                v[1] = static_cast<float>(acc[j][1]);
                v[2] = static_cast<float>(acc[j][2]);
                v[3] = static_cast<float>(acc[j][3]);
                __builtin_nontemporal_store(static_cast<v4f_dword_aligned>(v), reinterpret_cast<v4f_dword_aligned *>(dst));
            } else {
                dst[0] = static_cast<float>(acc[j][0]);
                if (floats > 1) dst[1] = static_cast<float>(acc[j][1]);
                if (floats > 2) dst[2] = static_cast<float>(acc[j][2]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// decoder on the float64 matrix cores
// ------------------------------------------------------------------------------------
// out = W (K x n) * Y (n x classes) with v_mfma_f64_16x16x4_f64, a workgroup of four waves per (group, tile of 64 vectors), the
// tiles those of sectors.h: the waves compute sixteen vectors each and exchange sixteen output rows at a time through LDS,
// from where they are stored as whole sectors.  Operand layout, lane l of the wave (c = l % 16, k = l / 16):
//   A: element (row c, k)    B: element (k, column c)    D: register t holds element (row 4 t + k, column c)
// so one 128-bit load of survivor 4 s + k gives the B operands of k-step s for four sets of columns, as in the encoder.
// NS k-steps: up to 4 NS survivors; their rows stay in registers for all ceil(K / 16) rounds.  Four waves per SIMD (79 to 125
// registers) hide the chain mask -> survivors -> rows and weights -> products; left to itself the compiler takes registers for
// two (K = 32, 36 groups of 32000 classes 99 us, with four 79).  An HBM stream next to float64 matrix issue (half of it at K = 32);
// two or four tiles to a workgroup that share their weights: 84 and 101 us where one each takes 81 (K = 20, 58 groups).
// coincide: up to sixteen queries, one of them on a worker's node.  If that worker answered, the query takes its row as it is,
// whatever the others returned, as in the tile kernels that serve those sizes too.  Beyond sixteen queries the other workers'
// rows count with weight zero, as in decode_kernel and in both class decisions there (their NaN or infinities then show), so
// that a group's answer does not depend on the size of the call.
// dynamic LDS: float stage[16][kStageRow] | double WdT[4 NS][KP] | alpha_s[K] | beta_s[N] | int F[N] | n | any hit | hit[64],
// KP = matrix_stride(K)
constexpr int kTileThreads = 256;
constexpr int kStageRow = 256 + 4;
// doubles between survivors in WdT: an odd number of 16-double lines, so that the four a wave reads lie in distinct banks
__host__ __device__ constexpr int matrix_stride(int K) { return 16 * (((K + 15) / 16) | 1); }

template <int NS>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(NS <= 9 ? 4 : 3))) void decode_matrix_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out, int32_t *__restrict__ status,
    int K, int N, int S, int64_t C, uint32_t per_row, int width, int halo, int sign_mode, int coincide, const Nodes nodes) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    extern __shared__ double lds_d[];
    const int KP = matrix_stride(K);
    float *stage = reinterpret_cast<float *>(lds_d);
    double *WdT = lds_d + 16 * kStageRow / 2;
    double *alpha_s = WdT + 4 * NS * KP;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = F + N;
    int *hit = n_sh + 2;                                      // survivor whose node query j is, or -1; n_sh[1]: any
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());
    const RowTile t = row_tile(blockIdx.x, per_row, width, halo, C);

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < 4 * NS * KP; e += kTileThreads) WdT[e] = 0.0;
    if (coincide && threadIdx.x < 64) hit[threadIdx.x] = -1;
    if (wv == 0) {
        const int n = survivors_from_mask(mask + t.g * N, N, F);
        if (lane == 0) {
            n_sh[0] = n;
            n_sh[1] = 0;
        }
    }
    __syncthreads();
    const int nF = *n_sh;
    const bool good = S < 0 ? nF >= 1 : nF == N - S;
    if (t.first && threadIdx.x == 0 && status != nullptr) status[t.g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    const int krow = lane >> 4;
    const int vec = wv * 16 + (lane & 15);                    // this lane's vector of the tile while computing
    const int c = t.column(vec);
    const float *pg = preds + static_cast<size_t>(t.g) * N * C + load_column(t, c, C);
    v4f y[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int r = 4 * s + krow;
        if (4 * s < nF)
            y[s] = __builtin_nontemporal_load(reinterpret_cast<const v4f_dword_aligned *>(
                pg + static_cast<size_t>(F[r < nF ? r : nF - 1]) * C));
    }
    for (int j = wv; coincide && j < K; j += kTileThreads / kWave)
        if (lane < nF && alpha_s[j] == beta_s[F[lane]]) {     // nodes are distinct: at most one lane
            hit[j] = lane;
            n_sh[1] = 1;
        }
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();
    const bool over = over_the_end(t, c);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (t.last && C % 4 != 0) y[s] = finish_vector(y[s], over, static_cast<int>(C % 4));
        if (4 * s + krow >= nF) y[s] = v4f(0.0f);             // no survivor: whatever the row holds counts for nothing
    }

    const bool hits = coincide && n_sh[1] != 0;
    float *og = out + static_cast<size_t>(t.g) * K * C + t.start;
    for (int j0 = 0; j0 < K; j0 += 16) {
        v4d acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = v4d{0.0, 0.0, 0.0, 0.0};
        const double *w = WdT + krow * KP + j0 + (lane & 15);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (4 * s < nF) {
                const double a = w[4 * s * KP];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, static_cast<double>(y[s][e]), acc[e], 0, 0, 0);
            }
        }
        if (j0 > 0) __syncthreads();                          // the rows of the round before are stored
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v4f v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = static_cast<float>(acc[e][r]);
            *reinterpret_cast<v4f *>(stage + (4 * r + krow) * kStageRow + 4 * vec) = v;
        }
        if (hits) {
            // behind this wave's own stores to the same columns; the row is read once more (kept, it costs all calls a fifth
            // of their time: 100 registers for 79)
            __builtin_amdgcn_wave_barrier();
            for (int r = krow; r < 16; r += 4) {
                const int h = hit[j0 + r];
                if (h < 0) continue;
                v4f v = *reinterpret_cast<const v4f_dword_aligned *>(preds + (static_cast<size_t>(t.g) * N + F[h]) * C +
                                                                     load_column(t, c, C));
                if (t.last && C % 4 != 0) v = finish_vector(v, over_the_end(t, c), static_cast<int>(C % 4));
                *reinterpret_cast<v4f *>(stage + r * kStageRow + 4 * vec) = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = j0 + 4 * wv + r;
            if (j < K) {
                float *row = og + static_cast<size_t>(j) * C;
                const int at = static_cast<int>(reinterpret_cast<uintptr_t>(row) / sizeof(float)) & (kSector - 1);
                store_sectors(row, *reinterpret_cast<const v4f *>(stage + (4 * wv + r) * kStageRow + 4 * lane), t.column(lane), at,
                              t);
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// decoder on the float64 matrix cores, short rows, more than sixteen queries
// ------------------------------------------------------------------------------------
// A wave per group, four to a workgroup, which walk the groups with the grid's stride: a tile of decode_matrix_kernel takes four
// waves and a set of weights, K |F| divisions, whatever the row's length.  Here T[i][j] = 1 / (alpha_j - beta_i), the same for all
// groups, is evaluated once per workgroup; the products of a wave are sums of T s_i y_i, s_i the alternating sign of survivor i, and
// the queries' denominators, one to a lane, divide them at the end.  A lane's D rows 4 t + k of consecutive k are neighbouring
// rows of out: sixteen lanes store vectors of one row, the next sixteen of the next.  Operand layout as in decode_matrix_kernel.
// R >= ceil(K / 16) rounds; rows of up to eight k-steps at a time stay in registers for all rounds and stripes of sixteen vectors
// come one after the other.  Float64 matrix issue and the chain of one group per wave at two waves a SIMD: 31 of 34 workers, K = 31, 14070
// groups of 36 classes 273 us with decode_kernel and 72 here (20 for the bytes); K = 48, 6851 of 60 307 and 78; K = 20, 487 of 40
// 13.4 and 8.2; K = 18, 7818 of 50 53 and 40.
// COINCIDE: some query has a worker's node.
// dynamic LDS: double T[N][short_stride(R)] | rden[4][16 R] | int F[4][64] | node[16 R].
constexpr int kShortWaves = 4;
constexpr int kShortClasses = 128;                            // two stripes
__host__ __device__ constexpr int short_stride(int R) { return 16 * (R | 1); }

template <int R, bool UNAL, bool COINCIDE>
__global__ __launch_bounds__(kShortWaves *kWave) __attribute__((amdgpu_waves_per_eu(2))) void decode_short_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out, int32_t *__restrict__ status,
    int64_t G, int K, int N, int S, int C, int sign_mode, const Nodes nodes) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int TS = short_stride(R), kSteps = 8;
    extern __shared__ double lds_d[];
    double *T = lds_d;
    double *rden = T + N * TS;
    int *F = reinterpret_cast<int *>(rden + kShortWaves * 16 * R);
    int *node = F + kShortWaves * kWave;                      // the worker whose node query j is, or -1
    const int lane = lane_id(), c = lane & 15, k = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());
    rden += wv * 16 * R;
    F += wv * kWave;

    if (COINCIDE) {
        if (static_cast<int>(threadIdx.x) < 16 * R) node[threadIdx.x] = -1;
        __syncthreads();
    }
    for (int e = threadIdx.x; e < N * 16 * R; e += kShortWaves * kWave) {
        const int i = e / (16 * R), j = e % (16 * R);
        const double d = j < K ? nodes.alpha[j] - nodes.beta[i] : 0.0;
        T[i * TS + j] = d != 0.0 ? 1.0 / d : 0.0;
        if (COINCIDE && j < K && d == 0.0) node[j] = i;       // nodes are distinct: one worker at most
    }
    __syncthreads();

    const int Cv = (C + 3) / 4;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * kShortWaves + wv; g < G; g += static_cast<int64_t>(gridDim.x) * kShortWaves) {
        __builtin_amdgcn_wave_barrier();                      // the group before has been through the list
        const bool in = lane < N && mask[g * N + lane] != 0;
        const unsigned long long bits = __ballot(in);
        const int nF = __popcll(bits);
        if (in) F[__popcll(bits & ((1ull << lane) - 1ull))] = lane;
        __builtin_amdgcn_wave_barrier();
        const bool good = S < 0 ? nF >= 1 : nF == N - S;
        if (lane == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
        if (!good) continue;
        const float *pg = preds + static_cast<size_t>(g) * N * C;
        float *og = out + static_cast<size_t>(g) * K * C;
        // A query on the node of a worker that answered: weight one for it, zero for the others (whose NaN or infinities show, as
        // in decode_kernel)
        const auto on_node = [&](int j) {
            const int i = node[j];
            return i >= 0 && ((bits >> i) & 1ull) != 0 ? i : -1;
        };
        int own[R];
        if (COINCIDE)
#pragma unroll
            for (int q = 0; q < R; ++q) own[q] = on_node(16 * q + c);
        for (int c0 = 0; c0 < Cv; c0 += 16) {
            const int cv = c0 + c;
            const int floats = cv >= Cv ? 0 : (UNAL && C - 4 * cv < 4 ? C - 4 * cv : 4);
            v4d acc[R][4];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[r][e] = v4d{0.0, 0.0, 0.0, 0.0};
            for (int s0 = 0; s0 < nF; s0 += 4 * kSteps) {
                v4f y[kSteps];
                int at[kSteps];
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
                    const int r = s0 + 4 * s + k;
                    y[s] = v4f(0.0f);
                    at[s] = F[r < nF ? r : nF - 1];
                    if (s0 + 4 * s < nF && r < nF && floats > 0)
                        y[s] = load_pred_vector<UNAL>(pg + static_cast<size_t>(at[s]) * C + 4 * cv, floats);
                }
                if (c0 == 0 && s0 == 0) {                     // while the first rows are on their way
                    double den = 0.0;
                    for (int r = 0; r < nF; ++r) {
                        const int i = __builtin_amdgcn_readfirstlane(F[r]);
                        const double t = T[i * TS + (lane < 16 * R ? lane : 0)];
                        den += ((sign_mode == APPROXIFER_SIGN_WORKER_INDEX ? i : r) & 1) ? -t : t;
                    }
                    if (lane < 16 * R) rden[lane] = COINCIDE && on_node(lane) >= 0 ? 1.0 : 1.0 / den;
                }
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
                    if (s0 + 4 * s < nF) {
                        const int r = s0 + 4 * s + k;
                        const int odd = (sign_mode == APPROXIFER_SIGN_WORKER_INDEX ? at[s] : r) & 1;
                        double a[R];
#pragma unroll
                        for (int q = 0; q < R; ++q) {
                            a[q] = T[at[s] * TS + 16 * q + c];
                            if (COINCIDE && own[q] >= 0) a[q] = at[s] != own[q] ? 0.0 : (odd ? -1.0 : 1.0);
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const double v = static_cast<double>(y[s][e]), b = odd ? -v : v;
#pragma unroll
                            for (int q = 0; q < R; ++q) acc[q][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b, acc[q][e], 0, 0, 0);
                        }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int j = 16 * q + 4 * t + k;
                    if (j < K && floats > 0) {
                        const double rd = rden[j];
                        v4f v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = static_cast<float>(acc[q][e][t] * rd);
                        float *dst = og + static_cast<size_t>(j) * C + 4 * cv;
                        if (!UNAL) {
                            __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(dst));
                        } else if (floats >= 4) {
                            __builtin_nontemporal_store(static_cast<v4f_dword_aligned>(v), reinterpret_cast<v4f_dword_aligned *>(dst));
                        } else {
                            dst[0] = v[0];
                            if (floats > 1) dst[1] = v[1];
                            if (floats > 2) dst[2] = v[2];
                        }
                    }
                }
        }
    }
}

// ------------------------------------------------------------------------------------
// fused decoder + top-1 kernel
// ------------------------------------------------------------------------------------
struct Best {
    double v;
    int i;
};
__device__ __forceinline__ bool better(double v, int i, const Best &b) { return v > b.v || (v == b.v && i < b.i); }

// One workgroup per group, one wave per quad of query rows.  A lane walks vector columns
// lane, lane+64, .. of its quad, decodes them in float64 exactly as contract_tile does and
// keeps the largest value (smallest class on equal values) per query row; a wavefront
// butterfly merges the 64 candidates; when the workgroup has more waves than quads, the waves
// of a quad split its columns and their winners are merged through LDS.  Nothing but [K] class
// indices (and scores) is written.
// dynamic LDS: as decode_kernel, then pad to 16 bytes | Best merged[KP][slices].
template <int VEC>
__global__ void decode_top1_kernel(const float *__restrict__ preds, const uint8_t *__restrict__ mask,
                                   int32_t *__restrict__ top1, float *__restrict__ score,
                                   int32_t *__restrict__ status, int K, int N, int S, int64_t C, int64_t Cv,
                                   int sign_mode, const Nodes nodes) {
    typedef typename PredVec<VEC>::type V;
    extern __shared__ double lds_d[];
    const int KP = round_up4(K);
    const int nF_cap = S < 0 ? N : N - S;          // S < 0: every group brings its own straggler count
    double *WdT = lds_d;
    double *alpha_s = WdT + nF_cap * KP;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = F + N;
    const int64_t g = blockIdx.x;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < nF_cap * KP; e += blockDim.x) WdT[e] = 0.0;
    if (wave_id() == 0) {
        const int n = survivors_from_mask(mask + g * N, N, F);
        if (lane_id() == 0) *n_sh = n;
    }
    __syncthreads();
    const int nF = *n_sh;
    const bool good = S < 0 ? nF >= 1 : nF == nF_cap;
    if (threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();

    const float *pg = preds + static_cast<size_t>(g) * N * C;
    const int lane = lane_id();
    const int KQ = KP / 4;
    const int nwaves = blockDim.x / kWave;
    const int slices = nwaves >= KQ ? nwaves / KQ : 1;          // waves that share one quad split its columns
    const int qwaves = nwaves >= KQ ? KQ : nwaves;              // quads processed concurrently
    const int slice = wave_id() / qwaves;
    Best *merged = reinterpret_cast<Best *>((reinterpret_cast<uintptr_t>(n_sh + 1) + 15) & ~static_cast<uintptr_t>(15));   // [KP][slices]
    for (int q = wave_id() % qwaves; q < KQ && slice < slices; q += qwaves) {
        Best best[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            best[jj].v = -__builtin_inf();
            best[jj].i = 0x7fffffff;
        }
        for (int64_t cv = static_cast<int64_t>(slice) * kWave + lane; cv < Cv; cv += static_cast<int64_t>(slices) * kWave) {
            double acc[4][VEC];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[jj][e] = 0.0;
            for (int r0 = 0; r0 < nF; r0 += kRowChunk) {
                V y[kRowChunk];
                load_row_chunk<VEC>(pg, F, nF, r0, C, cv, y);
#pragma unroll
                for (int u = 0; u < kRowChunk; ++u) {
                    if (r0 + u < nF) {
                        const double *w = WdT + (r0 + u) * KP + 4 * q;
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) {
                            const double wj = w[jj];
#pragma unroll
                            for (int e = 0; e < VEC; ++e)
                                acc[jj][e] = fma(wj, static_cast<double>(vec_get<VEC>(y[u], e)), acc[jj][e]);
                        }
                    }
                }
            }
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int idx = static_cast<int>(cv * VEC + e);
                    if (better(acc[jj][e], idx, best[jj])) {
                        best[jj].v = acc[jj][e];
                        best[jj].i = idx;
                    }
                }
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double ov = __shfl_xor(best[jj].v, off, kWave);
                const int oi = __shfl_xor(best[jj].i, off, kWave);
                if (better(ov, oi, best[jj])) {
                    best[jj].v = ov;
                    best[jj].i = oi;
                }
            }
            if (lane == 0) merged[(4 * q + jj) * slices + slice] = best[jj];
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < K; j += blockDim.x) {
        Best b = merged[j * slices];
        for (int sl = 1; sl < slices; ++sl) {
            const Best o = merged[j * slices + sl];
            if (better(o.v, o.i, b)) b = o;
        }
        top1[g * K + j] = b.i == 0x7fffffff ? 0 : b.i;
        if (score != nullptr) score[g * K + j] = static_cast<float>(b.v);
    }
}

// one step of a (value, class) maximum inside the 16-lane rows: larger value first, equal values: smaller class
template <int CTRL>
__device__ __forceinline__ void best_step(Best &b) {
    const double ov = dpp_exchange<CTRL>(b.v);
    const int oi = __builtin_amdgcn_update_dpp(0, b.i, CTRL, 0xF, 0xF, true);
    if (better(ov, oi, b)) {
        b.v = ov;
        b.i = oi;
    }
}

// ------------------------------------------------------------------------------------
// fused decoder + top-1, few groups of thousands of classes
// ------------------------------------------------------------------------------------
// A workgroup of up to sixteen waves per (group, QN queries).  Every lane walks vectors of four classes with the queries'
// accumulators and bests in registers; the next eight rows are on their way while the last eight are multiplied, across the end of
// a vector too.  The parts of a group read the same rows, from the caches.  What one CU has in flight bounds it (128 KB and 2 us a chunk
// of eight rows: 65 GB/s): K = 9, eight groups of 22613 classes, rows only 4-byte aligned, 72 us with a workgroup per quad of
// queries and 4-byte loads one chunk at a time, 26 this way; without a hint against the caches, and without loads for the rows
// that the last chunk lacks, which took 39.  A group's classes over several workgroups would need a place for their bests.
// dynamic LDS: double WdT[(N-S) QN] | alpha_s[K] | beta_s[N] | int F[N] | int n | pad to 16 bytes | Best merged[QN][waves].
constexpr int kSplitThreads = 1024;

template <int QN, bool UNAL>
__global__ __launch_bounds__(kSplitThreads) void decode_top1_split_kernel(const float *__restrict__ preds,
                                                                           const uint8_t *__restrict__ mask,
                                                                           int32_t *__restrict__ top1, float *__restrict__ score,
                                                                           int32_t *__restrict__ status, int K, int N, int S,
                                                                           int64_t C, int sign_mode, int parts, const Nodes nodes) {
    extern __shared__ double lds_d[];
    const int nF_cap = S < 0 ? N : N - S;
    double *WdT = lds_d;
    double *alpha_s = WdT + nF_cap * QN;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = F + N;
    Best *merged = reinterpret_cast<Best *>((reinterpret_cast<uintptr_t>(n_sh + 1) + 15) & ~static_cast<uintptr_t>(15));
    const int64_t g = blockIdx.x / parts;
    const int j0 = static_cast<int>(blockIdx.x - g * parts) * QN;
    const int own = K - j0 < QN ? K - j0 : QN;
    const int lane = lane_id();
    const int nwaves = blockDim.x / kWave;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < nF_cap * QN; e += blockDim.x) WdT[e] = 0.0;
    if (wave_id() == 0) {
        const int n = survivors_from_mask(mask + g * N, N, F);
        if (lane == 0) *n_sh = n;
    }
    __syncthreads();
    const int nF = __builtin_amdgcn_readfirstlane(*n_sh);
    const bool good = S < 0 ? nF >= 1 : nF == nF_cap;
    if (j0 == 0 && threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    const float *pgroup = preds + static_cast<size_t>(g) * N * C;
    const int Cv = static_cast<int>((C + 3) / 4);
    const auto floats_of = [&](int cv) { return UNAL && C - 4ll * cv < 4 ? static_cast<int>(C - 4ll * cv) : 4; };
    const auto load_rows = [&](int cv, int r0, v4f (&y)[kRowChunk]) {        // the parts of a group share them: no hint to the caches
        const int floats = floats_of(cv);
#pragma unroll
        for (int u = 0; u < kRowChunk; ++u) {
            if (r0 + u < nF) {
                const float *p = pgroup + static_cast<size_t>(__builtin_amdgcn_readfirstlane(F[r0 + u])) * C + 4ll * cv;
                if (!UNAL) {
                    y[u] = *reinterpret_cast<const v4f *>(p);
                } else if (floats >= 4) {
                    y[u] = *reinterpret_cast<const v4f_dword_aligned *>(p);
                } else {
                    y[u][0] = p[0];
                    if (floats > 1) y[u][1] = p[1];
                    if (floats > 2) y[u][2] = p[2];
                }
            }
        }
    };
    v4f ahead[kRowChunk];
    int cv = threadIdx.x;
    load_rows(cv < Cv ? cv : 0, 0, ahead);                  // in flight while the weights are evaluated
    decoder_weights(alpha_s + j0, beta_s, F, nF, own, QN, sign_mode, WdT);
    __syncthreads();

    Best best[QN];
#pragma unroll
    for (int j = 0; j < QN; ++j) {
        best[j].v = -__builtin_inf();
        best[j].i = 0x7fffffff;
    }
    for (; cv < Cv; cv += blockDim.x) {
        double acc[QN][4];
#pragma unroll
        for (int j = 0; j < QN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] = 0.0;
        for (int r0 = 0; r0 < nF; r0 += kRowChunk) {
            v4f y[kRowChunk];
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u) y[u] = ahead[u];
            const bool more = r0 + kRowChunk < nF;
            const int next = more ? cv : cv + static_cast<int>(blockDim.x);
            if (next < Cv) load_rows(next, more ? r0 + kRowChunk : 0, ahead);
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u) {
                if (r0 + u < nF) {
                    const double *w = WdT + (r0 + u) * QN;
                    const double y0 = y[u][0], y1 = y[u][1], y2 = y[u][2], y3 = y[u][3];
#pragma unroll
                    for (int j = 0; j < QN; ++j) {
                        const double wj = w[j];
                        acc[j][0] = fma(wj, y0, acc[j][0]);
                        acc[j][1] = fma(wj, y1, acc[j][1]);
                        acc[j][2] = fma(wj, y2, acc[j][2]);
                        acc[j][3] = fma(wj, y3, acc[j][3]);
                    }
                }
            }
        }
        const int floats = floats_of(cv);
#pragma unroll
        for (int j = 0; j < QN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < floats && better(acc[j][e], 4 * cv + e, best[j])) {
                    best[j].v = acc[j][e];
                    best[j].i = 4 * cv + e;
                }
    }
#pragma unroll
    for (int j = 0; j < QN; ++j) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double ov = __shfl_xor(best[j].v, off, kWave);
            const int oi = __shfl_xor(best[j].i, off, kWave);
            if (better(ov, oi, best[j])) {
                best[j].v = ov;
                best[j].i = oi;
            }
        }
        if (lane == 0) merged[j * nwaves + wave_id()] = best[j];
    }
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < own) {
        Best b = merged[threadIdx.x * nwaves];
        for (int w2 = 1; w2 < nwaves; ++w2) {
            const Best o = merged[threadIdx.x * nwaves + w2];
            if (better(o.v, o.i, b)) b = o;
        }
        const int64_t at = g * K + j0 + threadIdx.x;
        top1[at] = b.i == 0x7fffffff ? 0 : b.i;
        if (score != nullptr) score[at] = static_cast<float>(b.v);
    }
}

// ------------------------------------------------------------------------------------
// fused decoder + top-1 on the float64 matrix cores
// ------------------------------------------------------------------------------------
// One workgroup per group.  A wave takes stripes of sixteen vectors (64 classes), wave, wave + nwaves, .., multiplies as
// decode_matrix_kernel does and keeps, per lane, the best (value, class) so far of the 4 R queries whose rows it holds
// (R >= ceil(K / 16) rounds); the next stripe's rows are on their way meanwhile.  Nothing is stored until the end: sixteen
// lanes merge by DPP, the waves through LDS.  Ties: the smaller class index; NaN never wins.
// It is the chain load -> products -> best that bounds it, then float64 matrix issue (K = 32: see matrix_top1_shape).
// dynamic LDS: double WdT[4 NS][KP] | alpha_s[K] | beta_s[N] | Best merged[waves][16 R] | int F[N] | n
constexpr int top1_matrix_threads(int NS, int R) { return NS * R <= 8 ? 1024 : 512; }   // more registers: fewer waves

template <int NS, int R>
__global__ __launch_bounds__(top1_matrix_threads(NS, R)) void decode_top1_matrix_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, int32_t *__restrict__ top1, float *__restrict__ score,
    int32_t *__restrict__ status, int K, int N, int S, int64_t C, int sign_mode, const Nodes nodes) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    extern __shared__ double lds_d[];
    const int KP = matrix_stride(K);
    const int waves = blockDim.x / kWave;
    double *WdT = lds_d;
    double *alpha_s = WdT + 4 * NS * KP;
    double *beta_s = alpha_s + K;
    Best *merged = reinterpret_cast<Best *>(beta_s + N);
    int *F = reinterpret_cast<int *>(merged + waves * 16 * R);
    int *n_sh = F + N;
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int64_t g = blockIdx.x;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < 4 * NS * KP; e += blockDim.x) WdT[e] = 0.0;
    if (wv == 0) {
        const int n = survivors_from_mask(mask + g * N, N, F);
        if (lane == 0) *n_sh = n;
    }
    __syncthreads();
    const int nF = *n_sh;
    const bool good = S < 0 ? nF >= 1 : nF == N - S;
    if (threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    const int krow = lane >> 4, c = lane & 15;
    const float *pg = preds + static_cast<size_t>(g) * N * C;
    const float *rows[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) rows[s] = pg + static_cast<size_t>(F[4 * s + krow < nF ? 4 * s + krow : nF - 1]) * C;
    const int64_t stripes = (C + 63) / 64;
    v4f y[NS], next[NS];
    const auto load = [&](v4f(&to)[NS], int64_t stripe) {     // vectors past the row's end come from its last four columns
        const int64_t col = 64 * stripe + 4 * c;
        const int64_t at = col + 4 <= C ? col : C - 4;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (4 * s < nF) to[s] = __builtin_nontemporal_load(reinterpret_cast<const v4f_dword_aligned *>(rows[s] + at));
    };
    if (wv < stripes) load(y, wv);
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();

    Best best[R][4];
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) best[m][t] = Best{-__builtin_inf(), 0x7fffffff};
    for (int64_t stripe = wv; stripe < stripes; stripe += waves) {
        if (stripe + waves < stripes) load(next, stripe + waves);
        const int64_t col = 64 * stripe + 4 * c;
        const bool tail = stripe + 1 == stripes && C % 4 != 0;
        const bool over = col < C && col + 4 > C;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (tail) y[s] = finish_vector(y[s], over, static_cast<int>(C % 4));
            if (4 * s + krow >= nF) y[s] = v4f(0.0f);         // no survivor: whatever the row holds counts for nothing
        }
#pragma unroll
        for (int m = 0; m < R; ++m) {
            if (16 * m >= K) break;
            v4d acc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = v4d{0.0, 0.0, 0.0, 0.0};
            const double *w = WdT + krow * KP + 16 * m + c;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (4 * s < nF) {
                    const double a = w[4 * s * KP];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, static_cast<double>(y[s][e]), acc[e], 0, 0, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = col + e < C;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (in && acc[e][t] > best[m][t].v) best[m][t] = Best{acc[e][t], static_cast<int>(col + e)};
            }
        }
        if (stripe + waves < stripes) {
#pragma unroll
            for (int s = 0; s < NS; ++s) y[s] = next[s];
        }
    }
#pragma unroll
    for (int m = 0; m < R; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            Best b = best[m][t];
            best_step<kDppQuadXor1>(b);
            best_step<kDppQuadXor2>(b);
            best_step<kDppRowHalfMirror>(b);
            best_step<kDppRowMirror>(b);
            if (c == 0) merged[wv * 16 * R + 16 * m + 4 * t + krow] = b;
        }
    __syncthreads();
    for (int j = threadIdx.x; j < K; j += blockDim.x) {
        Best b = merged[j];
        for (int w = 1; w < waves; ++w) {
            const Best o = merged[w * 16 * R + j];
            if (better(o.v, o.i, b)) b = o;
        }
        top1[g * K + j] = b.i == 0x7fffffff ? 0 : b.i;
        if (score != nullptr) score[g * K + j] = static_cast<float>(b.v);
    }
}

// ------------------------------------------------------------------------------------
// fused decoder + top-1 with all K accumulator rows in one wave (K <= 16, up to 64 survivors)
// ------------------------------------------------------------------------------------
// One workgroup per group; its waves take the column tiles wave, wave + nwaves, .. and each keeps, per lane, the
// float64 accumulators of all K queries for four columns and the best (value, class) seen so far for every query.
// Nothing is stored inside the tile loop, so the next tile's loads are not held up by stores.  At the end a
// butterfly merges the lanes, LDS merges the waves.  Ties: the smaller class index.
// dynamic LDS: as decode_kernel, then pad to 16 bytes | Best merged[KP][nwaves].
template <int KQ, bool UNAL>
__global__ __launch_bounds__(256) void decode_top1_stream_kernel(const float *__restrict__ preds,
                                                                  const uint8_t *__restrict__ mask,
                                                                  int32_t *__restrict__ top1, float *__restrict__ score,
                                                                  int32_t *__restrict__ status, int K, int N, int S,
                                                                  int64_t C, int64_t Cv, int64_t ctiles, int sign_mode,
                                                                  const Nodes nodes) {
    constexpr int KP = 4 * KQ;
    extern __shared__ double lds_d[];
    const int nF_cap = S < 0 ? N : N - S;
    double *WdT = lds_d;
    double *alpha_s = WdT + nF_cap * KP;
    double *beta_s = alpha_s + K;
    int *F = reinterpret_cast<int *>(beta_s + N);
    int *n_sh = F + N;
    Best *merged = reinterpret_cast<Best *>((reinterpret_cast<uintptr_t>(n_sh + 1) + 15) & ~static_cast<uintptr_t>(15));
    const int64_t g = blockIdx.x;
    const int lane = lane_id();
    const int wv = wave_id();
    const int nwaves = blockDim.x / kWave;

    stage_nodes(nodes, K, N, alpha_s, beta_s);
    for (int e = threadIdx.x; e < nF_cap * KP; e += blockDim.x) WdT[e] = 0.0;
    if (wv == 0) {
        const int n = survivors_from_mask(mask + g * N, N, F);
        if (lane == 0) *n_sh = n;
    }
    __syncthreads();
    const int nF = *n_sh;
    const bool good = S < 0 ? nF >= 1 : nF == nF_cap;
    if (threadIdx.x == 0 && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    if (!good) return;

    const float *pgroup = preds + static_cast<size_t>(g) * N * C;
    // first tile of this wave: its first rows are in flight while the weights are evaluated
    v4f y[kRowChunk];
    {
        const int64_t cv_raw = static_cast<int64_t>(wv) * kColsPerTile + lane;
        const int64_t cv = cv_raw < Cv ? cv_raw : 0;
        const int floats = (UNAL && C - 4 * cv < 4) ? static_cast<int>(C - 4 * cv) : 4;
#pragma unroll
        for (int u = 0; u < kRowChunk; ++u)
            y[u] = load_pred_vector<UNAL>(pgroup + 4 * cv + static_cast<size_t>(F[u < nF ? u : nF - 1]) * C, floats);
    }
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();

    Best best[KP];
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        best[j].v = -__builtin_inf();
        best[j].i = 0x7fffffff;
    }
    for (int64_t ct = wv; ct < ctiles; ct += nwaves) {
        const int64_t cv_raw = ct * kColsPerTile + lane;
        const bool ok = cv_raw < Cv;
        const int64_t cv = ok ? cv_raw : 0;
        const int floats = (UNAL && C - 4 * cv < 4) ? static_cast<int>(C - 4 * cv) : 4;
        const float *pg = pgroup + 4 * cv;
        double acc[KP][4];
#pragma unroll
        for (int j = 0; j < KP; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] = 0.0;
        for (int r0 = 0; r0 < nF; r0 += kRowChunk) {
            if (r0 > 0 || ct != wv) {
#pragma unroll
                for (int u = 0; u < kRowChunk; ++u)
                    y[u] = load_pred_vector<UNAL>(pg + static_cast<size_t>(F[r0 + u < nF ? r0 + u : nF - 1]) * C, floats);
            }
#pragma unroll
            for (int u = 0; u < kRowChunk; ++u) {
                if (r0 + u < nF) {
                    const double *w = WdT + (r0 + u) * KP;
                    const double y0 = y[u][0], y1 = y[u][1], y2 = y[u][2], y3 = y[u][3];
#pragma unroll
                    for (int j = 0; j < KP; ++j) {
                        const double wj = w[j];
                        acc[j][0] = fma(wj, y0, acc[j][0]);
                        acc[j][1] = fma(wj, y1, acc[j][1]);
                        acc[j][2] = fma(wj, y2, acc[j][2]);
                        acc[j][3] = fma(wj, y3, acc[j][3]);
                    }
                }
            }
        }
        if (ok) {
#pragma unroll
            for (int j = 0; j < KP; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int idx = static_cast<int>(cv * 4 + e);
                    if (e < floats && better(acc[j][e], idx, best[j])) {
                        best[j].v = acc[j][e];
                        best[j].i = idx;
                    }
                }
        }
    }
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        // the wave's best: four DPP steps inside each row of 16 lanes, then the four rows by v_readlane
        best_step<kDppQuadXor1>(best[j]);
        best_step<kDppQuadXor2>(best[j]);
        best_step<kDppRowHalfMirror>(best[j]);
        best_step<kDppRowMirror>(best[j]);
        Best b = best[j];
        b.v = read_lane(best[j].v, 0);
        b.i = __builtin_amdgcn_readlane(best[j].i, 0);
#pragma unroll
        for (int row = 1; row < 4; ++row) {
            const double ov = read_lane(best[j].v, 16 * row);
            const int oi = __builtin_amdgcn_readlane(best[j].i, 16 * row);
            if (better(ov, oi, b)) {
                b.v = ov;
                b.i = oi;
            }
        }
        if (lane == 0) merged[j * nwaves + wv] = b;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < K; j += blockDim.x) {
        Best b = merged[j * nwaves];
        for (int w2 = 1; w2 < nwaves; ++w2) {
            const Best o = merged[j * nwaves + w2];
            if (better(o.v, o.i, b)) b = o;
        }
        top1[g * K + j] = b.i == 0x7fffffff ? 0 : b.i;
        if (score != nullptr) score[g * K + j] = static_cast<float>(b.v);
    }
}

// ------------------------------------------------------------------------------------
// what the row kernels below share: a 16-lane row works on one group, N <= 64
// ------------------------------------------------------------------------------------
// T[i][j] = 1 / (alpha_j - beta_i), row stride KP, zero for j >= K and where the two nodes are one; hit[j] = the worker
// whose node is query node j, or -1, hit[KP] = whether there is one.  By the whole workgroup, one entry per thread from
// nodes that begin() has sent for; ends with a barrier.
template <int KP>
struct NodeTable {
    double alpha, beta;                                     // of entry threadIdx.x
    __device__ __forceinline__ void begin(const Nodes &nodes, int K, int N, int *hit) {
        const int e = threadIdx.x < N * KP ? threadIdx.x : 0;
        alpha = nodes.alpha[e % KP < K ? e % KP : 0];
        beta = nodes.beta[e / KP];
        if (threadIdx.x <= KP) hit[threadIdx.x] = threadIdx.x < KP ? -1 : 0;
    }
    // unit: also T[N + i][j] = 1 where the two nodes are one, else 0
    __device__ __forceinline__ void finish(const Nodes &nodes, int K, int N, double *T, int *hit, bool unit) {
        __syncthreads();
        for (int e = threadIdx.x; e < N * KP; e += blockDim.x) {
            const int i = e / KP, j = e % KP;
            if (e >= static_cast<int>(blockDim.x)) {
                alpha = nodes.alpha[j < K ? j : 0];
                beta = nodes.beta[i];
            }
            const double d = alpha - beta;
            const bool same = j < K && d == 0.0;
            if (same) {                                     // nodes are distinct: one worker at most
                hit[j] = i;
                hit[KP] = 1;
            }
            T[e] = (j < K && !same) ? 1.0 / d : 0.0;
            if (unit) T[N * KP + e] = same ? 1.0 : 0.0;
        }
        __syncthreads();
    }
};
// The mask row of this lane's group, byte lane % 16 + 16 p in b[p]; lanes past N load byte 0 (four loads that nothing
// waits for, instead of four branches with a load in each).
struct MaskBytes {
    uint8_t b[4];
};
__device__ __forceinline__ MaskBytes load_mask_row(const uint8_t *__restrict__ mask_row, int N) {
    MaskBytes r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int i = p * kRowLanes + static_cast<int>(threadIdx.x % kRowLanes);
        r.b[p] = mask_row[i < N ? i : 0];
    }
    return r;
}
// Bit i of the result: worker i of this lane's group answered.
__device__ __forceinline__ unsigned long long row_survivors(const MaskBytes &r, int N) {
    unsigned long long m = 0ull;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        m |= ((__ballot(r.b[p] != 0) >> (lane_id() & 48)) & 0xffffull) << (p * kRowLanes);
    return N < 64 ? m & ((1ull << N) - 1ull) : m;
}
// Bit i, for a survivor i: its term of the decoder carries a minus sign.
__device__ __forceinline__ unsigned long long minus_signs(unsigned long long m, int sign_mode) {
    if (sign_mode != APPROXIFER_SIGN_SURVIVOR_RANK) return 0xaaaaaaaaaaaaaaaaull;       // an odd index
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) m ^= m << s;           // bit i: an odd number of survivors up to and including i
    return ~m;
}

// Lists the survivors of this row's group, visible to the row after the wave barrier at the end: F[0 .. nF) ascending, and
// every entry behind them names the first survivor, so that a pass over the list never names a worker that did not
// answer.  (No survivor: zeros, which nobody may follow.)
__device__ __forceinline__ void list_survivors(unsigned long long m, uint8_t *F) {
    const int lane = static_cast<int>(threadIdx.x % kRowLanes);
    list_first(m, F, lane);
    list_ranks(m, F, lane);
    __builtin_amdgcn_wave_barrier();
}
// The most survivors that any row of this wave has.
__device__ __forceinline__ int most_survivors_of_wave(int nF) {
    return max(max(__builtin_amdgcn_readlane(nF, 0), __builtin_amdgcn_readlane(nF, 16)),
               max(__builtin_amdgcn_readlane(nF, 32), __builtin_amdgcn_readlane(nF, 48)));
}

// ------------------------------------------------------------------------------------
// small classes: a 16-lane row per group
// ------------------------------------------------------------------------------------
// K <= 32 queries, N <= 64 workers, C <= 16 classes: the image-classification operating points (K = 8..12, one to three
// stragglers, ten classes) and the text shapes (two classes).  A group is a few hundred bytes; what its decode took was
// launch and barrier latency with a workgroup per group, and the issue slots of the weights, two divisions and a
// reduction per entry, with a wave per group.  Here a group is one 16-lane row, lane = class, sixteen groups to a
// workgroup, and no weights are formed.  T[i][j] = 1 / (alpha_j - beta_i) depends on the nodes only and is evaluated
// once per workgroup, while the loads are in flight; with s_i = the alternating sign of worker i, 0 if it did not answer,
//     out[j][c] = (sum_i T[i][j] s_i y_ic) / (sum_i T[i][j] s_i).
// Lane j holds T[i][j], from where the numerators of all classes take it inside the multiply-add (row_outer), and sums
// the denominator of query j.  The pass goes over the list of survivors: rows of missing workers are not read, and the
// predictions wait for the mask.
// A query node that is a worker's node has T = 0 there; if the worker answered, the query takes its row as it is.
// 16384 groups of K = 8, N = 9, ten classes, top-1: 13.1 us a kernel with a wave per group, 7.2 us this way.
// QS = 4: four rows share a group, a quarter of its queries each.  While the launch does not fill the chip it takes as
// long as one row's chain (K <= 8, up to 1024 groups: 2.9 us split, 3.2 unsplit, 2.9 with a wave per group that forms
// weights; K = 9..16 3.7, 4.5 and 4.0 us); beyond, the unsplit rows do more with what they load (K <= 8, 4096 to 8191
// groups 3.6 us, 5.1 split).
constexpr int64_t kRowsSplitGroups = 2048;
constexpr int kRowGroups = 16;
constexpr int kRowChunkSmall = 16;      // prediction rows in flight
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

template <bool TOP1, int KP, int QS>
__global__ __launch_bounds__(kRowGroups *kRowLanes) void decode_rows_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out,
    int32_t *__restrict__ top1, float *__restrict__ score, int32_t *__restrict__ status, int64_t G, int K, int N,
    int S, int C, int sign_mode, const Nodes nodes) {
    constexpr int KQ = KP / QS;                              // queries of a row: j0 ..
    constexpr int kRegs = (KQ + kRowLanes - 1) / kRowLanes;  // T and denominators of query j0 + lane + 16 h in register h
    extern __shared__ __align__(16) double T[];             // [N][KP] | int hit[KP] | int any_hit | pad | uint8 F[16][80]
    int *hit = reinterpret_cast<int *>(T + N * KP);
    const int c = threadIdx.x % kRowLanes;
    const int row = threadIdx.x / kRowLanes;
    uint8_t *F = reinterpret_cast<uint8_t *>(hit + KP + 4) + row * kListBytes;
    const int64_t g_raw = static_cast<int64_t>(blockIdx.x) * (kRowGroups / QS) + row / QS;
    const int j0 = row % QS * KQ;
    const bool here = g_raw < G;
    const int64_t g = here ? g_raw : G - 1;                 // rows past the last group work on it and store nothing

    const MaskBytes answered = load_mask_row(mask + g * N, N);
    NodeTable<KP> table;
    table.begin(nodes, K, N, hit);
    const unsigned long long m = row_survivors(answered, N);
    const int nF = static_cast<int>(__popcll(m));
    const bool good = S < 0 ? nF >= 1 : nF == N - S;
    if (c == 0 && row % QS == 0 && here && status != nullptr) status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    list_survivors(m, F);
    const int rows = S < 0 ? most_survivors_of_wave(nF) : N - S;
    const uint32_t by_index = sign_mode == APPROXIFER_SIGN_SURVIVOR_RANK ? 0u : 1u;
    const float *pg = preds + static_cast<size_t>(g) * N * C + (c < C ? c : 0);

    v4u f;
    float y[kRowChunkSmall];
    const auto load_chunk = [&](int r0) {
        f = *reinterpret_cast<const v4u *>(F + r0);
#pragma unroll
        for (int u = 0; u < kRowChunkSmall; ++u) y[u] = 0.0f;
#pragma unroll
        for (int q = 0; q < kRowChunkSmall; q += 4) {
            if (r0 + q < rows && nF > 0) {
#pragma unroll
                for (int u = q; u < q + 4; ++u) y[u] = pg[static_cast<int>((f[u / 4] >> (8 * (u % 4))) & 0xffu) * C];
            }
        }
    };
    load_chunk(0);
    table.finish(nodes, K, N, T, hit, false);               // while the first predictions are on their way

    double acc[KQ], den[kRegs];
#pragma unroll
    for (int j = 0; j < KQ; ++j) acc[j] = 0.0;
#pragma unroll
    for (int h = 0; h < kRegs; ++h) den[h] = 0.0;
    for (int r0 = 0; r0 < rows; r0 += kRowChunkSmall) {
        if (r0 > 0) load_chunk(r0);
#pragma unroll
        for (int u = 0; u < kRowChunkSmall; ++u) {
            if (r0 + u < rows) {
                const uint32_t w = (f[u / 4] >> (8 * (u % 4))) & 0xffu;
                const uint32_t there = r0 + u < nF ? ~0u : 0u;              // rows of the wave may differ in nF
                const uint32_t flip = ((w & by_index) | (u & 1u & ~by_index)) << 31;
                const double sy = static_cast<double>(__uint_as_float((__float_as_uint(y[u]) ^ flip) & there));
                const double s = __hiloint2double(static_cast<int>((0x3ff00000u ^ flip) & there), 0);
                double t[kRegs];
#pragma unroll
                for (int h = 0; h < kRegs; ++h) {
                    const int j = h * kRowLanes + c;
                    t[h] = T[w * KP + j0 + (j < KQ ? j : 0)];
                    den[h] = fma(s, t[h], den[h]);
                }
                row_outer<0, 0, (KQ < kRowLanes ? KQ : kRowLanes)>(acc, t[0], sy);
                if constexpr (kRegs > 1) row_outer<kRowLanes, 0, KQ - kRowLanes>(acc, t[1], sy);
            }
        }
    }
#pragma unroll
    for (int h = 0; h < kRegs; ++h) den[h] = 1.0 / den[h];
#pragma unroll
    for (int j = 0; j < KQ; ++j) acc[j] *= row_bcast_dyn(den[j / kRowLanes], j % kRowLanes);
    if (hit[KP] != 0) {
#pragma unroll
        for (int j = 0; j < KQ; ++j) {
            const int h = hit[j0 + j];
            if (h >= 0 && ((m >> h) & 1ull) != 0ull) acc[j] = static_cast<double>(pg[h * C]);
        }
    }
    if (!TOP1) {
        float *og = out + static_cast<size_t>(g) * K * C + c;
        if (here && good && c < C) {
#pragma unroll
            for (int j = 0; j < KQ; ++j)
                if (j0 + j < K) og[(j0 + j) * C] = static_cast<float>(acc[j]);
        }
        return;
    }
    // largest value of each query, smallest class on equal values, kept by the lane of the query.  NaN loses to any number;
    // a query without any value above -inf gets class 0 and that class's value.  Lanes past the last class hold -inf too,
    // so that they win nothing.
    int best_c[kRegs];
    double best_v[kRegs];
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
        const double v = c < C ? acc[j] : -__builtin_inf();
        double b = v;
        b = __builtin_fmax(b, dpp_exchange<kDppQuadXor1>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppQuadXor2>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppRowHalfMirror>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppRowMirror>(b));
        const uint32_t who = static_cast<uint32_t>(__ballot(v == b && v > -__builtin_inf()) >> (lane_id() & 48)) & 0xffffu;
        const double first = row_bcast<0>(v);
        if (c == j % kRowLanes) {
            best_v[j / kRowLanes] = who != 0u ? b : first;
            best_c[j / kRowLanes] = who != 0u ? __ffs(who) - 1 : 0;
        }
    }
#pragma unroll
    for (int h = 0; h < kRegs; ++h) {
        const int j = h * kRowLanes + c;
        if (here && good && j < KQ && j0 + j < K) {
            top1[g * K + j0 + j] = best_c[h];
            if (score != nullptr) score[g * K + j0 + j] = static_cast<float>(best_v[h]);
        }
    }
}

// ------------------------------------------------------------------------------------
// more classes: a 16-lane row per (group, sixteen vectors of four classes)
// ------------------------------------------------------------------------------------
// The same for K <= 16, N <= 64 and more than sixteen classes: a lane owns four neighbouring classes, a tile is 64 classes
// of a group, and a workgroup takes sixteen consecutive tiles of the batch, so that a row end leaves at most fifteen
// lanes idle where a wave per (group, 256 classes) left up to 63 (100 classes: 7 of 32 against 39 of 64).  A lane has CHUNK
// rows in flight; everything else, T above all, is evaluated while the mask is on its way.
// UNAL: rows are only 4-byte aligned; the lane with a row's last partial vector moves it float by float.
// 4096 groups of K = 8, 8 of 12 workers, 100 classes: 8.6 us with a wave per 256 classes, 7.1 us this way; 65536 groups
// of 40 classes 88 and 40 us; 512 groups of K = 12, 12 of 20 workers, 1000 classes 13.4 and 11.3 us.
// Which calls come here: tiles_shape.  K = 9..12 with twelve rows in flight (two waves to a SIMD) is faster while one
// round of workgroups holds the launch (8192 tiles), slower after that: 512 groups of 1000 classes 11.1 us against 12.9
// with eight rows (three waves), 1024 groups of 4000 classes 76.8 against 71.7.
constexpr int64_t kTilesOneRound = 8192;

// The worker whose node is a query node (hit[]), if it answered, else -1.
__device__ __forceinline__ int own_worker(int h, unsigned long long m) { return h >= 0 && ((m >> h) & 1ull) != 0ull ? h : -1; }
// This lane's query's column of the table.  A query whose node is that of a worker that answered takes the worker's row as it
// is: its column is the unit vector kept behind T.  (To load the row again at the end cost a round trip to memory for each
// such query: K = 13, 16 of 27 workers, three such queries, 317 groups of 808 classes 18.9 us, 13.0 this way.)
template <int KP>
__device__ __forceinline__ const double *query_column(const double *T, const int *hit, int N, unsigned long long m) {
    const int c = threadIdx.x % kRowLanes < KP ? threadIdx.x % kRowLanes : 0;
    return T + c + (own_worker(hit[c], m) >= 0 ? N * KP : 0);
}

// acc[e][j] = sum over the survivors i of T[i][j] s_i y_ie, this lane's four classes e of the row at pg + class; den: in
// lane j the denominator of query j.  rows: the most survivors that any row of the wave may have.  A row past its last
// survivor repeats its first (S < 0: with factor 0); the values of a bad row are not used, and one without survivors
// reads nothing.
template <int KP, int CHUNK, bool UNAL>
__device__ __forceinline__ void tile_sums(const float *__restrict__ pg, int64_t C, int floats, const uint8_t *F, int nF,
                                          int rows, bool varies, unsigned long long minus, const double *column,
                                          double (&acc)[4][KP], double &den) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < KP; ++j) acc[e][j] = 0.0;
    den = 0.0;
#pragma unroll 1
    for (int r0 = 0; r0 < rows; r0 += CHUNK) {
        v4f y[CHUNK];
        int w[CHUNK];
#pragma unroll
        for (int u = 0; u < CHUNK; ++u) {
            w[u] = F[r0 + u];
            y[u] = v4f(0.0f);
        }
        if (nF > 0) {
#pragma unroll
            for (int u = 0; u < CHUNK; ++u) y[u] = load_pred_vector<UNAL>(pg + static_cast<size_t>(w[u]) * C, floats);
        }
#pragma unroll
        for (int u = 0; u < CHUNK; ++u) {
            if (r0 + u < rows) {
                const uint32_t flip = (static_cast<uint32_t>(minus >> w[u]) & 1u) << 31;
                double s = __hiloint2double(static_cast<int>(0x3ff00000u ^ flip), 0);
                if (varies && r0 + u >= nF) {
                    s = 0.0;
                    y[u] = v4f(0.0f);
                }
                const double t = column[w[u] * KP];
                den = fma(s, t, den);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    row_outer<0, 0, KP>(acc[e], t, static_cast<double>(__uint_as_float(__float_as_uint(y[u][e]) ^ flip)));
            }
        }
    }
}
template <int KP, int CHUNK, bool UNAL>
__global__ __launch_bounds__(kRowGroups *kRowLanes) void decode_tiles_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, float *__restrict__ out,
    int32_t *__restrict__ status, int64_t tiles, uint32_t chunks, int K, int N, int S, int64_t C, int sign_mode,
    const Nodes nodes) {
    extern __shared__ double T[];                           // [2 N][KP] | int hit[KP] | int any_hit | pad | uint8 F[16][80]
    int *hit = reinterpret_cast<int *>(T + 2 * N * KP);
    const int c = threadIdx.x % kRowLanes;
    const int row = threadIdx.x / kRowLanes;
    uint8_t *F = reinterpret_cast<uint8_t *>(hit + KP + 4) + row * kListBytes;
    const int64_t tile_raw = static_cast<int64_t>(blockIdx.x) * kRowGroups + row;
    const bool here = tile_raw < tiles;
    const int64_t tile = here ? tile_raw : tiles - 1;
    const int64_t g = tiles <= 0xffffffffLL ? static_cast<uint32_t>(tile) / chunks : tile / chunks;
    const uint32_t chunk = static_cast<uint32_t>(tile - g * chunks);

    const MaskBytes answered = load_mask_row(mask + g * N, N);
    NodeTable<KP> table;
    table.begin(nodes, K, N, hit);
    table.finish(nodes, K, N, T, hit, true);
    const unsigned long long m = row_survivors(answered, N), minus = minus_signs(m, sign_mode);
    const int nF = static_cast<int>(__popcll(m));
    const bool good = S < 0 ? nF >= 1 : nF == N - S;
    if (c == 0 && here && chunk == 0 && status != nullptr)
        status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    list_survivors(m, F);
    const int rows = S < 0 ? most_survivors_of_wave(nF) : N - S;
    const double *column = query_column<KP>(T, hit, N, m);

    const int64_t col = (static_cast<int64_t>(chunk) * kRowLanes + c) * 4;
    const bool ok = col < C;
    const int floats = UNAL && ok && C - col < 4 ? static_cast<int>(C - col) : 4;
    const float *pg = preds + static_cast<size_t>(g) * N * C + (ok ? col : 0);
    double acc[4][KP], den;
    tile_sums<KP, CHUNK, UNAL>(pg, C, floats, F, nF, rows, S < 0, minus, column, acc, den);
    den = 1.0 / den;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        const double d = row_bcast_dyn(den, j);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e][j] *= d;
    }
    if (hit[KP] != 0) {                                          // another worker's NaN or infinity does not reach such a query
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const int h = own_worker(hit[j], m);
            const double sum = (acc[0][j] + acc[1][j]) + (acc[2][j] + acc[3][j]);
            if (good && h >= 0 && !(__builtin_fabs(sum) < __builtin_inf())) {
                const v4f yh = load_pred_vector<UNAL>(pg + static_cast<size_t>(h) * C, floats);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e][j] = static_cast<double>(yh[e]);
            }
        }
    }
    float *og = out + static_cast<size_t>(g) * K * C + col;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        v4f f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = static_cast<float>(acc[e][j]);
        if (here && good && ok && j < K) {
            float *dst = og + static_cast<size_t>(j) * C;
            if (!UNAL) {
                __builtin_nontemporal_store(f, reinterpret_cast<v4f *>(dst));
            } else if (floats >= 4) {
                __builtin_nontemporal_store(static_cast<v4f_dword_aligned>(f), reinterpret_cast<v4f_dword_aligned *>(dst));
            } else {
                dst[0] = f[0];
                if (floats > 1) dst[1] = f[1];
                if (floats > 2) dst[2] = f[2];
            }
        }
    }
}

// The class decision over the same tiles: R = 1, 2, 4, 8 or 16 rows of a workgroup share a group, row q taking the tiles
// q, q + R, ..; a lane keeps the best (value, class) of every query over its tiles, the lanes of a row meet by DPP, the
// rows of a group in LDS.  4096 groups of 100 classes (K = 8, 8 of 12 workers): 18.0 us with a workgroup per group, 7.9 us
// this way; 512 groups of 1000 classes (K = 12): 16.5 and 12.9 us; 16384 groups of 40: 53 and 12.
template <int KP, int CHUNK, bool UNAL>
__global__ __launch_bounds__(kRowGroups *kRowLanes) void decode_top1_tiles_kernel(
    const float *__restrict__ preds, const uint8_t *__restrict__ mask, int32_t *__restrict__ top1,
    float *__restrict__ score, int32_t *__restrict__ status, int64_t G, uint32_t chunks, int R, int K, int N, int S,
    int64_t C, int sign_mode, const Nodes nodes) {
    extern __shared__ double T[];                           // [2 N][KP] | best values [16][KP] | int best classes [16][KP]
    double *best_v = T + 2 * N * KP;                            // | int hit[KP] | int any_hit | pad | uint8 F[16][80]
    int *best_c = reinterpret_cast<int *>(best_v + kRowGroups * KP);
    int *hit = best_c + kRowGroups * KP;
    const int c = threadIdx.x % kRowLanes;
    const int row = threadIdx.x / kRowLanes;
    uint8_t *F = reinterpret_cast<uint8_t *>(hit + KP + 4) + row * kListBytes;
    const int64_t g_raw = static_cast<int64_t>(blockIdx.x) * (kRowGroups / R) + row / R;
    const bool here = g_raw < G;
    const int64_t g = here ? g_raw : G - 1;

    const MaskBytes answered = load_mask_row(mask + g * N, N);
    NodeTable<KP> table;
    table.begin(nodes, K, N, hit);
    table.finish(nodes, K, N, T, hit, true);
    const unsigned long long m = row_survivors(answered, N), minus = minus_signs(m, sign_mode);
    const int nF = static_cast<int>(__popcll(m));
    const bool good = S < 0 ? nF >= 1 : nF == N - S;
    if (c == 0 && here && row % R == 0 && status != nullptr)
        status[g] = good ? APPROXIFER_GROUP_OK : APPROXIFER_GROUP_BAD_MASK;
    list_survivors(m, F);
    const int rows = S < 0 ? most_survivors_of_wave(nF) : N - S;
    const double *column = query_column<KP>(T, hit, N, m);

    double bv[KP];
    int bc[KP];
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        bv[j] = -__builtin_inf();
        bc[j] = 0x7fffffff;
    }
#pragma unroll 1
    for (uint32_t base = 0; base < chunks; base += R) {     // every row goes round as often as the others
        const int64_t col = (static_cast<int64_t>(base + row % R) * kRowLanes + c) * 4;
        const bool ok = col < C;
        const int floats = ok ? (C - col < 4 ? static_cast<int>(C - col) : 4) : 0;
        const float *pg = preds + static_cast<size_t>(g) * N * C + (ok ? col : 0);
        double acc[4][KP], den;
        tile_sums<KP, CHUNK, UNAL>(pg, C, UNAL && ok ? floats : 4, F, nF, rows, S < 0, minus, column, acc, den);
        den = 1.0 / den;
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const double d = row_bcast_dyn(den, j);
            double v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[e][j] * d;
            if (hit[KP] != 0) {                                  // another worker's NaN or infinity does not reach such a query
                const int h = own_worker(hit[j], m);
                const double sum = (v[0] + v[1]) + (v[2] + v[3]);
                if (good && h >= 0 && !(__builtin_fabs(sum) < __builtin_inf())) {
                    const v4f yh = load_pred_vector<UNAL>(pg + static_cast<size_t>(h) * C, UNAL && ok ? floats : 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = static_cast<double>(yh[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {                   // ascending classes: the first of equal values stays
                const bool take = e < floats && v[e] > bv[j];
                bv[j] = take ? v[e] : bv[j];
                bc[j] = take ? static_cast<int>(col) + e : bc[j];
            }
        }
    }
    // largest value of the row, smallest class on equal values; lane j keeps query j's
    double mine_v = -__builtin_inf();
    int mine_c = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        double b = bv[j];
        b = __builtin_fmax(b, dpp_exchange<kDppQuadXor1>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppQuadXor2>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppRowHalfMirror>(b));
        b = __builtin_fmax(b, dpp_exchange<kDppRowMirror>(b));
        int i = bv[j] == b ? bc[j] : 0x7fffffff;
        i = min(i, __builtin_amdgcn_update_dpp(0, i, kDppQuadXor1, 0xF, 0xF, true));
        i = min(i, __builtin_amdgcn_update_dpp(0, i, kDppQuadXor2, 0xF, 0xF, true));
        i = min(i, __builtin_amdgcn_update_dpp(0, i, kDppRowHalfMirror, 0xF, 0xF, true));
        i = min(i, __builtin_amdgcn_update_dpp(0, i, kDppRowMirror, 0xF, 0xF, true));
        if (c == j) {
            mine_v = b;
            mine_c = i;
        }
    }
    if (R > 1) {
        if (c < KP) {
            best_v[row * KP + c] = mine_v;
            best_c[row * KP + c] = mine_c;
        }
        __syncthreads();
        if (row % R != 0) return;
        for (int q = 1; q < R && c < KP; ++q) {
            const double v = best_v[(row + q) * KP + c];
            const int i = best_c[(row + q) * KP + c];
            if (v > mine_v || (v == mine_v && i < mine_c)) {
                mine_v = v;
                mine_c = i;
            }
        }
    }
    if (here && good && c < K) {
        top1[g * K + c] = mine_c == 0x7fffffff ? 0 : mine_c;             // nothing above -inf: class 0
        if (score != nullptr) score[g * K + c] = static_cast<float>(mine_v);
    }
}

// ------------------------------------------------------------------------------------
// wait rule: arrival times -> survivor mask
// ------------------------------------------------------------------------------------
// One wave per group, four groups per workgroup; a lane owns workers lane and lane + 64.  The rank of a
// worker is the number of workers that answer before it (equal times: smaller index first), counted
// against the group's times broadcast from the wave's LDS; the wait_for lowest ranks are the survivors.
constexpr int kWaitGroups = 4;

__global__ __launch_bounds__(kWaitGroups *kWave) void wait_mask_kernel(const float *__restrict__ arrival,
                                                                         uint8_t *__restrict__ mask,
                                                                         int32_t *__restrict__ count, int64_t G, int N,
                                                                         int wait_for) {
    __shared__ float t_s[kWaitGroups][APPROXIFER_MAX_N];
    const int lane = lane_id();
    const int wv = wave_id();
    const int64_t g = static_cast<int64_t>(blockIdx.x) * kWaitGroups + wv;
    if (g >= G) return;
    float *t = t_s[wv];
    const float never = __builtin_inff();
    float mine[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int i = lane + p * kWave;
        float v = never;
        if (i < N) {
            v = arrival[g * N + i];
            if (!(fabsf(v) < never)) v = never;           // NaN and both infinities: never answers
            t[i] = v;
        }
        mine[p] = v;
    }
    __builtin_amdgcn_wave_barrier();
    int total = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int i = lane + p * kWave;
        int rank = 0;
#pragma unroll 8
        for (int o = 0; o < N; ++o) {
            const float other = t[o];
            rank += (other < mine[p] || (other == mine[p] && o < i)) ? 1 : 0;
        }
        const bool in = i < N && mine[p] < never && rank < wait_for;
        if (i < N) mask[g * N + i] = in ? 1 : 0;
        total += __popcll(__ballot(in));
    }
    if (lane == 0 && count != nullptr) count[g] = total;
}

// ------------------------------------------------------------------------------------
// top-1 of an already decoded tensor
// ------------------------------------------------------------------------------------
// LPR lanes per row of [rows][C] float32 (a wave for long rows, sixteen lanes for rows of up to 32 classes, so that a
// wave takes four rows of a ten-class output instead of idling 54 lanes on one): largest value, smallest class on
// equal values (NaN never wins; a row of NaNs gives class 0).  Four waves per workgroup.
constexpr int kArgmaxWaves = 4;

template <int LPR>
__global__ __launch_bounds__(kArgmaxWaves *kWave) void argmax_rows_kernel(const float *__restrict__ values,
                                                                           int32_t *__restrict__ top1,
                                                                           float *__restrict__ score, int64_t rows,
                                                                           int64_t C) {
    constexpr int kRowsPerWave = kWave / LPR;
    const int lane = lane_id();
    const int64_t row = (static_cast<int64_t>(blockIdx.x) * kArgmaxWaves + wave_id()) * kRowsPerWave + lane / LPR;
    const bool live = row < rows;
    const float *v = values + (live ? row : 0) * C;
    float bv = -__builtin_inff();
    int bi = 0x7fffffff;
    for (int64_t c = lane % LPR; c < C; c += LPR) {
        const float x = v[c];
        if (x > bv) {                                       // ascending c: the first occurrence stays
            bv = x;
            bi = static_cast<int>(c);
        }
    }
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off, kWave);
        const int oi = __shfl_xor(bi, off, kWave);
        if (ov > bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
        }
    }
    if (live && lane % LPR == 0) {
        const bool none = bi == 0x7fffffff;                 // every value NaN or -inf
        top1[row] = none ? 0 : bi;
        if (score != nullptr) score[row] = none ? v[0] : bv;
    }
}

bool rows_shape(int K, int N, int64_t C) { return K <= 32 && N <= kWave && C <= kRowLanes; }

// Whether decode_tiles_kernel decodes the call (K <= 16, N <= 64).  Over 1900 shapes of 2 to 16 queries and 17 to 32000
// classes, inputs in rotation, it was 2 to 11 % slower than a wave per 256 classes where it took them all; it gains
//  - where most of that wave's lanes lie past the end of the row and groups abound: up to 100 classes, from 2048 groups
//    (K = 8, 4096 groups of 100 classes 8.7 -> 7.2 us; 65536 groups of 40 classes 88 -> 40 us);
//  - for K = 9..16 and a known number of survivors while one round of workgroups holds the launch (512 groups of K = 12,
//    1000 classes 13.4 -> 10.7 us): 5 % on average from 1024 tiles on, where it loses 9 % beyond 8192 (84 groups of K = 9,
//    16000 classes 21.4 and 26.7 us); up to K = 12 for up to twelve survivors, which one pass takes (13 to 16: 13 % slower);
//  - rows that are only 4-byte aligned are loaded float by float at their ends, by every sixteenth lane instead of every
//    64th: worth it for up to 80 classes and many groups only (K = 4, 1024 groups of 1003 classes 10.1 and 14.5 us).
bool tiles_shape(int K, int N, int S, int64_t C, int64_t G, bool vec4) {
    if (K > 16 || N > kWave) return false;
    const int64_t vectors = (C + 3) / 4;
    if (!vec4) return vectors <= 20 && G * K >= 32768;
    const int64_t tiles = G * ((vectors + kRowLanes - 1) / kRowLanes);
    if (vectors <= 25 && G >= 2048) return true;
    return K > 8 && S >= 0 && (K > 12 || N - S <= 12) && tiles >= 1024 && tiles <= kTilesOneRound;
}
// Whether decode_matrix_kernel decodes the call (more than eight queries, up to 64 workers, more than sixteen classes).  Its
// tile takes four waves, whatever the row's length, so it is not for many groups of short rows; times without and with it:
//  - K > 16: from 96 classes on (K = 32, 1170 groups of 1001 classes 241 and 96 us, 1171 of 1000 145 and 92), up to kShortClasses against
//    decode_short_kernel while tiles are few (100 classes: K = 21, 975 groups 17.6 there and 13.7 in decode_short_kernel, K = 21, 443 of
//    122 13.3 and 17.9; K = 40, 6009 of 100 171 and 105), and in calls of few tiles (84 classes: K = 31, seven groups
//    9.8 and 12.8; up to 64 even with it, K = 32, 250 of 32 10.0 and 11.1, K = 20, 36 of 20 9.1 and 8.6); fewer than 64 classes in rows that are only 4-byte aligned from 25 queries or 33 survivors on (K = 21, 28 survivors, 33 classes, three
//    groups 8.9 and 9.3; K = 18, 40 survivors, 19 classes, two groups 12.5 and 11.2);
//  - K = 9..16 in rows that are only 4-byte aligned: from 96 classes on (K = 16, 2341 groups of 1001 classes 101 and 74 us, 78
//    groups 15.9 and 7.7), with K = 9..11, which leave a third of the products' rows empty, up to 4096 tiles (K = 9, 832 groups of
//    1001 classes 27.9 and 24.1, 4162 groups 98 and 103), up to 2048 with sixteen survivors or fewer (K = 10, ten survivors, 796 of
//    1027 25.1 and 28.4) and not between one and a half rounds of the chip and two and a half where two tiles take a row of little
//    more than one (K = 9, 1039 of 253 14.5 and 20.8), and in calls of few tiles (K = 12, 50 classes, 208 groups 10.9 and 5.8 us, 2083
//    groups 16.0 and 14.3);
//  - K = 9..16 otherwise in calls of few tiles, whose time is one workgroup's chain: its weights are four waves' work (K = 12, ten
//    groups of 1000 classes 7.2 and 5.3 us, 104 groups 7.1 and 7.0, 156 of 4000 classes 14.3 and 16.1; K = 13, 24 groups of 4000
//    classes 8.1 and 6.3, 144 groups 20.4 and 17.2, 2884 of 1000 classes 68 and 83).
bool matrix_shape(int K, int N, int S, int64_t C, int64_t G, bool vec4) {
    if (K <= 8 || N > kWave || C <= kRowLanes) return false;
    const int64_t tiles = G * ((C + 239) / 240);
    const int survivors = S < 0 ? N : N - S;
    if (K > 16) return C > kShortClasses || (C >= 96 && tiles <= 500) || (tiles <= 400 && (vec4 || K > 24 || C >= 64 || survivors > 32));
    if (!vec4 && C >= 96) {
        const SectorTiles t = sector_tiles(G, C, kTileHalo);
        return K > 11 || (t.total <= (survivors > 16 ? 4096 : 2048) && (t.width >= 4 * 38 || t.per_row == 1 || t.total <= 1536 || t.total > 2560));
    }
    if (!vec4) return tiles <= (C >= 48 ? 2048 : 400);
    return tiles <= (K > 12 ? 1024 : 400) || (K > 12 && C >= 96 && tiles <= 4096 && !tiles_shape(K, N, S, C, G, vec4));
}
// Whether decode_top1_tiles_kernel decides the call: all of them (0.76 of the time of a workgroup per group over 1600
// shapes), but for long rows that are only 4-byte aligned with few queries to make up for their ends (K = 3, 7900 groups of
// 750 classes 48.8 and 79.5 us; K = 8 from 4096 groups on 3 to 8 % slower).
bool top1_tiles_shape(int K, int N, int64_t C, int64_t G, bool vec4) {
    if (K > 16 || N > kWave) return false;
    return vec4 || C <= 128 || K > 8 || (K > 4 && G < 4096);
}

int64_t top1_split_waves(int64_t C) { return std::min<int64_t>((C + 4 * kWave - 1) / (4 * kWave), kSplitThreads / kWave); }

// Queries to a workgroup of decode_top1_split_kernel, 0: not the call's kernel.  For up to 512 quads of queries, whose other kernels
// leave most of the chip idle and wait for one chunk of rows after the other.  Times without and with it, 680 calls:
//  - rows of whole vectors: K > 16 always (K = 28, 15 groups of 2520 classes 38.6 and 11.7 us, K = 64, 19 of 3844 345 and 55, K = 24,
//    20 classes, 36 quads 15.3 and 8.4); K = 9..16 from 384 classes on (one group of 21844 32 and 25; K = 16, 40 of 288 7.7 and
//    8.0), up to 240 quads where they are shorter than 2000 (K = 14, 77 of 688 8.3 and 9.8); K <= 8 from 256 (K = 6, 4 of 6176 14.0 and
//    9.7), shorter than 4096 while a CU has one workgroup or two queries to each (K = 4, 336 of 2156 11.1 and 16.0, 449 of 420 6.5 and 8.3);
//  - rows that are only 4-byte aligned: always from 4096 classes on (K = 9, 8 groups of 22613 72 and 26); K > 32 always (214
//    classes, 32 quads 54 and 18), K = 17..32 from 64 (874 classes, 8 quads 22.6 and 12.0; 43 classes, 180 quads 11.0 and 11.4);
//    K = 9..16 from 1900 up to 200 quads (2125 classes, 90 quads 12.6 and 9.6; 1597, 396 quads 14.1 and 17.2; 511, one group 7.7
//    and 10.6), K <= 8 from 100, while a CU has one workgroup or the waves are few (K = 8, 152 of 1178 18.5 and 11.3; K = 5, 163 of
//    2351 14.0 and 17.1).
// Two queries to a workgroup while that gives each CU one workgroup, or all of them together 1600 waves (K = 20, 76 of 260 10.0 with
// four and 8.1; K = 7, 184 of 372 7.6 and 6.1; K = 20, 35 of 2168 12.9 and 18.9); with more than 12000 classes up to 176, from
// where on the rows that the parts read again cost more (K = 28, 11 of 23540 59 and 48; K = 12, 39 of 25640 40 and 48).
int top1_split(int K, int64_t C, int64_t G, bool vec4) {
    const int64_t quads = G * ((K + 3) / 4), pairs = G * ((K + 1) / 2), waves = top1_split_waves(C);
    if (quads > 512 || C <= kRowLanes || C > 0x7fffffff) return 0;
    const int queries = K <= 2 || pairs <= (C <= 12000 ? 256 : 176) || pairs * waves <= 1600 ? 2 : 4;
    const int64_t blocks = G * ((K + queries - 1) / queries);
    bool faster;
    if (K > 32) faster = true;
    else if (K > 16) faster = vec4 || C >= 64;
    else if (K > 8) faster = vec4 ? C >= 384 && (C >= 2000 || quads <= 240) : C >= 4093 || (C >= 1900 && quads <= 200);
    else if (vec4) faster = C >= 256 && (C >= 4096 || blocks <= 256 || queries == 2);
    else faster = C >= 100 && (C >= 4093 || blocks <= 256 || queries == 2 || blocks * waves <= 2000);
    return faster ? queries : 0;
}

template <bool TOP1, int KP, int QS>
int run_rows_shape(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_top1, float *d_score,
                   int32_t *d_status, int64_t G, int K, int N, int S, int64_t C, const Nodes &nodes, int sign_mode,
                   hipStream_t stream) {
    constexpr int kGroups = kRowGroups / QS;
    const int64_t blocks = (G + kGroups - 1) / kGroups;
    if (blocks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    return launch_status(launch_kernel(decode_rows_kernel<TOP1, KP, QS>, dim3(static_cast<unsigned>(blocks)),
                                       dim3(kRowGroups * kRowLanes),
                                       sizeof(double) * N * KP + sizeof(int) * (KP + 4) + kRowGroups * kListBytes, stream, d_preds,
                                       d_mask, d_out, d_top1, d_score, d_status, G, K, N, S, static_cast<int>(C), sign_mode,
                                       nodes));
}

template <bool TOP1>
int run_rows(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_top1, float *d_score, int32_t *d_status,
             int64_t G, int K, int N, int S, int64_t C, const Nodes &nodes, int sign_mode, hipStream_t stream) {
#define APPROXIFER_ROWS(KP)                                                                                            \
    (G <= kRowsSplitGroups ? run_rows_shape<TOP1, KP, 4>(d_preds, d_mask, d_out, d_top1, d_score, d_status, G, K, N, S, C,    \
                                                         nodes, sign_mode, stream)                                      \
                           : run_rows_shape<TOP1, KP, 1>(d_preds, d_mask, d_out, d_top1, d_score, d_status, G, K, N, S, C,    \
                                                         nodes, sign_mode, stream))
    switch ((K + 3) / 4) {
        case 1: return APPROXIFER_ROWS(4);
        case 2: return APPROXIFER_ROWS(8);
        case 3: return APPROXIFER_ROWS(12);
        case 4: return APPROXIFER_ROWS(16);
        case 5:
        case 6: return APPROXIFER_ROWS(24);
        default: return APPROXIFER_ROWS(32);
    }
#undef APPROXIFER_ROWS
}

bool nodes_coincide(const Nodes &nodes, int K, int N) {
    int any = 0;
    for (int j = 0; j < K; ++j)
        for (int i = 0; i < N; ++i) any |= nodes.alpha[j] == nodes.beta[i];
    return any != 0;
}

template <int NS>
int run_matrix(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_status, int64_t G, int K, int N, int S,
               int64_t C, const Nodes &nodes, int sign_mode, hipStream_t stream) {
    const int halo = whole_sectors(d_out, C) ? 0 : kTileHalo;
    const SectorTiles t = sector_tiles(G, C, halo);
    if (t.total > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const size_t lds = sizeof(float) * 16 * kStageRow + sizeof(double) * (static_cast<size_t>(4 * NS) * matrix_stride(K) + K + N) +
                       sizeof(int) * (static_cast<size_t>(N) + 2 + APPROXIFER_MAX_K);
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(decode_matrix_kernel<NS>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(decode_matrix_kernel<NS>, dim3(static_cast<unsigned>(t.total)),
                                       dim3(kTileThreads), lds, stream, d_preds, d_mask, d_out, d_status, K, N, S, C,
                                       static_cast<uint32_t>(t.per_row), t.width, halo, sign_mode,
                                       K <= 16 && nodes_coincide(nodes, K, N) ? 1 : 0, nodes));
}

template <int R>
int run_short(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_status, int64_t G, int K, int N, int S,
              int64_t C, bool vec4, const Nodes &nodes, int sign_mode, hipStream_t stream) {
    const int64_t blocks = std::min<int64_t>((G + kShortWaves - 1) / kShortWaves, 1024);
    const size_t lds = sizeof(double) * (static_cast<size_t>(N) * short_stride(R) + kShortWaves * 16 * R) +
                       sizeof(int) * (kShortWaves * kWave + 16 * R);
    const auto run = [&](auto *kernel) {
        return launch_status(launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kShortWaves * kWave), lds, stream, d_preds,
                                           d_mask, d_out, d_status, G, K, N, S, static_cast<int>(C), sign_mode, nodes));
    };
    if (nodes_coincide(nodes, K, N)) return run(vec4 ? decode_short_kernel<R, false, true> : decode_short_kernel<R, true, true>);
    return run(vec4 ? decode_short_kernel<R, false, false> : decode_short_kernel<R, true, false>);
}

// Whether decode_top1_matrix_kernel decides the call (more than eight queries, up to 64 workers, more than sixteen classes) that
// top1_split leaves.  Times without and with it, over 5000 calls:
//  - K = 9..16 in rows that are only 4-byte aligned: always (0.2 to 0.96 of the time; K = 12, 6243 groups of 1001 classes 204 and 96, 206
//    of 101 15.5 and 5.6);
//  - K = 9..16 otherwise: against tiles that share a workgroup's sixteen rows of lanes.  Up to 256 classes in few groups (K = 16,
//    4000 of 40 7.0 and 8.3, 20000 of 96 1.39 times); longer rows up to 24 survivors always (K = 12, 6250 of 1000 133 and 98), with more
//    in one round of workgroups (G <= 256) and, up to 36 survivors, in many (N = 40, 384 to 1024 groups of 1000 classes 1.1 to 1.4 times);
//  - K = 17..27 in whole vectors from 256 groups on (K = 17, 147 of 1000 17.8 and 20.8); K = 32, 2341 groups of 1001 classes 644 and 172,
//    23205 of 101 1238 and 304, 2343 of 1000 292 and 170;
//  - K > 32: few groups of few classes stay with a wave per quad of queries (K = 48, 128 groups of 64 classes 1.24 times, of 33 1.44,
//    500 of 33 25.5 and 30.5 us).
// K <= 8 leaves half of the products' rows empty (K = 8, 9375 of 1000 100 and 117).  Up to sixteen queries the other kernels
// hand on the row of a worker whose node a query has, whatever the other workers returned; calls with such nodes stay there.
bool top1_matrix_shape(int K, int N, int S, int64_t C, int64_t G, bool vec4, const Nodes &nodes) {
    if (K <= 8 || N > kWave || C <= kRowLanes) return false;
    if (K <= 16) {
        const int64_t stripes = (C + 63) / 64;
        const int survivors = S < 0 ? N : N - S;
        const bool faster = !vec4 || (stripes <= 4 ? G * (stripes + 1) <= 5120 : survivors <= 24 || G <= 256 || (survivors <= 36 && G > 1024));
        return faster && !nodes_coincide(nodes, K, N);
    }
    if (K > 32 && (vec4 ? C <= 400 && G <= 256 : C <= 64 && G <= 512)) return false;
    return !vec4 || K >= 28 || G >= 256;
}

template <int NS, int R>
int run_top1_matrix_shape(const float *d_preds, const uint8_t *d_mask, int32_t *d_top1, float *d_score, int32_t *d_status,
                          int64_t G, int K, int N, int S, int64_t C, const Nodes &nodes, int sign_mode, hipStream_t stream) {
    if (G > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    // a wave per stripe, up to four; more where there are few groups to fill the chip with, but all of them in one round: up to
    // 256 groups the kernel's most, up to 512 half of it (K = 12, 500 groups of 1000 classes, eight waves 0.77 and sixteen 1.33 of the
    // other kernel's time; N = 40, 400 groups, four waves 0.92 and eight 1.16).  Up to 512 groups at least four waves: the weights
    // are the whole workgroup's work (beyond 48 queries up to 1023)
    constexpr int most = top1_matrix_threads(NS, R) / kWave;
    const int64_t stripes = (C + 63) / 64;
    int64_t waves = G <= 256 ? most : G <= 512 ? most / 2 : 4;
    if (waves > stripes) waves = G > (K > 48 ? 1023 : 512) || stripes > 4 ? stripes : 4;
    const size_t lds = sizeof(double) * (static_cast<size_t>(4 * NS) * matrix_stride(K) + K + N) + sizeof(Best) * waves * 16 * R +
                       sizeof(int) * (static_cast<size_t>(N) + 2);
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(decode_top1_matrix_kernel<NS, R>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(decode_top1_matrix_kernel<NS, R>, dim3(static_cast<unsigned>(G)),
                                       dim3(static_cast<unsigned>(waves) * kWave), lds, stream, d_preds, d_mask, d_top1, d_score,
                                       d_status, K, N, S, C, sign_mode, nodes));
}

int run_top1_matrix(const float *d_preds, const uint8_t *d_mask, int32_t *d_top1, float *d_score, int32_t *d_status, int64_t G,
                    int K, int N, int S, int64_t C, const Nodes &nodes, int sign_mode, hipStream_t stream) {
    const int steps = ((S < 0 ? N : N - S) + 3) / 4;
#define APPROXIFER_TOP1_MATRIX(NS)                                                                                      \
    (K <= 16 ? run_top1_matrix_shape<NS, 1>(d_preds, d_mask, d_top1, d_score, d_status, G, K, N, S, C, nodes, sign_mode, stream) \
     : K <= 32                                                                                                           \
         ? run_top1_matrix_shape<NS, 2>(d_preds, d_mask, d_top1, d_score, d_status, G, K, N, S, C, nodes, sign_mode, stream) \
         : run_top1_matrix_shape<NS, 4>(d_preds, d_mask, d_top1, d_score, d_status, G, K, N, S, C, nodes, sign_mode, stream))
    if (steps <= 4) return APPROXIFER_TOP1_MATRIX(4);
    if (steps <= 6) return APPROXIFER_TOP1_MATRIX(6);
    if (steps <= 9) return APPROXIFER_TOP1_MATRIX(9);
    return APPROXIFER_TOP1_MATRIX(16);
#undef APPROXIFER_TOP1_MATRIX
}

}  // namespace

int launch_decode(const float *d_preds, const uint8_t *d_mask, float *d_out, int32_t *d_status, int64_t G, int K,
                  int N, int S, int64_t C, const Nodes &nodes, int sign_mode, hipStream_t stream) {
    if (rows_shape(K, N, C))
        return run_rows<false>(d_preds, d_mask, d_out, nullptr, nullptr, d_status, G, K, N, S, C, nodes, sign_mode, stream);
    const int KP = (K + 3) & ~3;
    const bool vec4 = (C % 4 == 0) && aligned16(d_preds) && aligned16(d_out);
    if (matrix_shape(K, N, S, C, G, vec4)) {
        const int steps = ((S < 0 ? N : N - S) + 3) / 4;
        if (steps <= 4) return run_matrix<4>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, nodes, sign_mode, stream);
        if (steps <= 6) return run_matrix<6>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, nodes, sign_mode, stream);
        if (steps <= 9) return run_matrix<9>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, nodes, sign_mode, stream);
        if (steps <= 12) return run_matrix<12>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, nodes, sign_mode, stream);
        return run_matrix<16>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, nodes, sign_mode, stream);
    }
    // what matrix_shape leaves of these, otherwise a workgroup per group with a wave for every four queries (figures at the kernel);
    // beyond two stripes the third is mostly empty (K = 28, 2362 groups of 132 classes 46.6 and 55.4 us)
    if (K > 16 && N <= kWave && C <= kShortClasses)
        return K <= 32 ? run_short<2>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, vec4, nodes, sign_mode, stream)
                       : run_short<4>(d_preds, d_mask, d_out, d_status, G, K, N, S, C, vec4, nodes, sign_mode, stream);
    const int64_t Cv = vec4 ? C / 4 : C;
    const int64_t ctiles = (Cv + kColsPerTile - 1) / kColsPerTile;
    const int64_t blocks = G * ctiles;
    if (blocks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    int waves = KP / 4;
    if (waves > 4) waves = 4;
    const size_t lds = sizeof(double) * (static_cast<size_t>(S < 0 ? N : N - S) * KP + K + N) + sizeof(int) * (static_cast<size_t>(N) + 2);
    if (tiles_shape(K, N, S, C, G, vec4)) {
        const int64_t chunks = ((C + 3) / 4 + kRowLanes - 1) / kRowLanes;
        const int64_t tiles = G * chunks;
        const int64_t tblocks = (tiles + kRowGroups - 1) / kRowGroups;
        if (tblocks > 0x7fffffffLL || chunks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
        const dim3 tgrid(static_cast<unsigned>(tblocks)), tblock(kRowGroups * kRowLanes);
#define APPROXIFER_TILES(KPV, CHUNK, UNAL)                                                                             \
    launch_status(launch_kernel(decode_tiles_kernel<KPV, CHUNK, UNAL>, tgrid, tblock,                                   \
                                sizeof(double) * 2 * N * KPV + sizeof(int) * (KPV + 4) + kRowGroups * kListBytes, stream, d_preds,  \
                                d_mask, d_out, d_status, tiles, static_cast<uint32_t>(chunks), K, N, S, C, sign_mode, nodes))
        switch (KP / 4) {
            case 1: return vec4 ? APPROXIFER_TILES(4, 8, false) : APPROXIFER_TILES(4, 8, true);
            case 2: return vec4 ? APPROXIFER_TILES(8, 8, false) : APPROXIFER_TILES(8, 8, true);
            case 3:
                if (!vec4) return APPROXIFER_TILES(12, 8, true);
                return tiles <= kTilesOneRound ? APPROXIFER_TILES(12, 12, false) : APPROXIFER_TILES(12, 8, false);
            default: return vec4 ? APPROXIFER_TILES(16, 8, false) : APPROXIFER_TILES(16, 8, true);
        }
#undef APPROXIFER_TILES
    }
    // all other calls of up to 16 queries and 64 survivors: one wave per 256 classes with all K accumulator rows (capping
    // its residency as in the encoder changes nothing: 4 to 12 waves per CU +-3 %)
    const int most_survivors = S < 0 ? N : N - S;
    if (K <= 16 && most_survivors <= 64 && C >= 4) {
        const int64_t sCv = (C + 3) / 4;                  // counts a partial last vector
        const int64_t stiles = (sCv + kColsPerTile - 1) / kColsPerTile;
        if (G * stiles > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
        const dim3 sgrid(static_cast<unsigned>(G * stiles)), sblock(kWave);
#define APPROXIFER_STREAM(KQ, UNAL)                                                                                    \
    launch_status(launch_kernel(decode_stream_kernel<KQ, UNAL>, sgrid, sblock, lds, stream, d_preds, d_mask, d_out,       \
                                d_status, K, N, S, C, sCv, stiles, sign_mode, nodes))
        switch (KP / 4) {
            case 1: return vec4 ? APPROXIFER_STREAM(1, false) : APPROXIFER_STREAM(1, true);
            case 2: return vec4 ? APPROXIFER_STREAM(2, false) : APPROXIFER_STREAM(2, true);
            case 3: return vec4 ? APPROXIFER_STREAM(3, false) : APPROXIFER_STREAM(3, true);
            default: return vec4 ? APPROXIFER_STREAM(4, false) : APPROXIFER_STREAM(4, true);
        }
#undef APPROXIFER_STREAM
    }
    const dim3 grid(static_cast<unsigned>(blocks)), block(waves * kWave);
    if (lds > 64 * 1024) {   // only K = 64 with more than 127 survivors; gfx950 has 160 KB of LDS per CU
        const void *fn = vec4 ? reinterpret_cast<const void *>(decode_kernel<4>)
                              : reinterpret_cast<const void *>(decode_kernel<1>);
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
            return APPROXIFER_ERR_LAUNCH;
    }
    return launch_status(launch_kernel(vec4 ? decode_kernel<4> : decode_kernel<1>, grid, block, lds, stream, d_preds, d_mask,
                                       d_out, d_status, K, N, S, C, Cv, ctiles, sign_mode, nodes));
}

int launch_decode_top1(const float *d_preds, const uint8_t *d_mask, int32_t *d_top1, float *d_score,
                       int32_t *d_status, int64_t G, int K, int N, int S, int64_t C, const Nodes &nodes,
                       int sign_mode, hipStream_t stream) {
    if (rows_shape(K, N, C))
        return run_rows<true>(d_preds, d_mask, nullptr, d_top1, d_score, d_status, G, K, N, S, C, nodes, sign_mode, stream);
    const int KP = (K + 3) & ~3;
    const bool vec4 = (C % 4 == 0) && aligned16(d_preds);
    const int64_t Cv = vec4 ? C / 4 : C;
    if (G > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const int KQ = KP / 4;
    const int split = top1_split(K, C, G, vec4);
    // up to sixteen queries the tile kernel hands on the row of a worker whose node a query has; calls that it used to serve stay
    if (split > 0 && (K > 16 || N > kWave || C >= 4093 || !nodes_coincide(nodes, K, N))) {
        const int parts = (K + split - 1) / split;
        const int64_t waves = top1_split_waves(C);
        const size_t slds = sizeof(double) * (static_cast<size_t>(S < 0 ? N : N - S) * split + K + N) +
                            sizeof(int) * (static_cast<size_t>(N) + 1) + 16 + sizeof(Best) * split * waves;
        const dim3 sgrid(static_cast<unsigned>(G * parts)), sblock(static_cast<unsigned>(waves) * kWave);
#define APPROXIFER_TOP1_SPLIT(QN, UNAL)                                                                                 \
    launch_status(launch_kernel(decode_top1_split_kernel<QN, UNAL>, sgrid, sblock, slds, stream, d_preds, d_mask, d_top1,  \
                                d_score, d_status, K, N, S, C, sign_mode, parts, nodes))
        if (split == 2) return vec4 ? APPROXIFER_TOP1_SPLIT(2, false) : APPROXIFER_TOP1_SPLIT(2, true);
        return vec4 ? APPROXIFER_TOP1_SPLIT(4, false) : APPROXIFER_TOP1_SPLIT(4, true);
#undef APPROXIFER_TOP1_SPLIT
    }
    if (top1_matrix_shape(K, N, S, C, G, vec4, nodes))
        return run_top1_matrix(d_preds, d_mask, d_top1, d_score, d_status, G, K, N, S, C, nodes, sign_mode, stream);
    if (top1_tiles_shape(K, N, C, G, vec4)) {
        const int64_t chunks = ((C + 3) / 4 + kRowLanes - 1) / kRowLanes;
        int R = 1;
        while (R < kRowGroups && R < chunks) R *= 2;
        const dim3 tgrid(static_cast<unsigned>((G + kRowGroups / R - 1) / (kRowGroups / R))), tblock(kRowGroups * kRowLanes);
#define APPROXIFER_TOP1_TILES(KPV, CHUNK, UNAL)                                                                        \
    launch_status(launch_kernel(decode_top1_tiles_kernel<KPV, CHUNK, UNAL>, tgrid, tblock,                              \
                                sizeof(double) * (2 * N + kRowGroups) * KPV + sizeof(int) * (kRowGroups * KPV + KPV + 4) +   \
                                    kRowGroups * kListBytes,                                                                 \
                                stream, d_preds, d_mask, d_top1, d_score, d_status, G, static_cast<uint32_t>(chunks), R, K, \
                                N, S, C, sign_mode, nodes))
        switch (KQ) {
            case 1: return vec4 ? APPROXIFER_TOP1_TILES(4, 8, false) : APPROXIFER_TOP1_TILES(4, 8, true);
            case 2: return vec4 ? APPROXIFER_TOP1_TILES(8, 8, false) : APPROXIFER_TOP1_TILES(8, 8, true);
            case 3: return vec4 ? APPROXIFER_TOP1_TILES(12, 8, false) : APPROXIFER_TOP1_TILES(12, 8, true);
            default: return vec4 ? APPROXIFER_TOP1_TILES(16, 8, false) : APPROXIFER_TOP1_TILES(16, 8, true);
        }
#undef APPROXIFER_TOP1_TILES
    }
    // K <= 16, up to 64 survivors: a workgroup per group whose waves keep all K accumulator rows
    if (K <= 16 && (S < 0 ? N : N - S) <= 64 && C >= 4) {
        const int64_t sCv = (C + 3) / 4;
        const int64_t stiles = (sCv + kColsPerTile - 1) / kColsPerTile;
        const int nwaves = stiles < 4 ? static_cast<int>(stiles) : 4;
        size_t slds = sizeof(double) * (static_cast<size_t>(S < 0 ? N : N - S) * KP + K + N) + sizeof(int) * (static_cast<size_t>(N) + 3);
        slds += 16 + sizeof(double) * 2 * static_cast<size_t>(KP) * nwaves;
        const dim3 sgrid(static_cast<unsigned>(G)), sblock(nwaves * kWave);
#define APPROXIFER_TOP1_STREAM(KQV, UNAL)                                                                              \
    launch_status(launch_kernel(decode_top1_stream_kernel<KQV, UNAL>, sgrid, sblock, slds, stream, d_preds, d_mask,       \
                                d_top1, d_score, d_status, K, N, S, C, sCv, stiles, sign_mode, nodes))
        switch (KQ) {
            case 1: return vec4 ? APPROXIFER_TOP1_STREAM(1, false) : APPROXIFER_TOP1_STREAM(1, true);
            case 2: return vec4 ? APPROXIFER_TOP1_STREAM(2, false) : APPROXIFER_TOP1_STREAM(2, true);
            case 3: return vec4 ? APPROXIFER_TOP1_STREAM(3, false) : APPROXIFER_TOP1_STREAM(3, true);
            default: return vec4 ? APPROXIFER_TOP1_STREAM(4, false) : APPROXIFER_TOP1_STREAM(4, true);
        }
#undef APPROXIFER_TOP1_STREAM
    }
    int slices = static_cast<int>((Cv + kWave - 1) / kWave);     // column slices worth a wave of their own
    const int most = G >= 512 ? 4 : 16;                          // few groups: all sixteen waves of a workgroup
    if (slices > most) slices = most;
    if (slices * KQ > 16) slices = 16 / KQ;
    if (slices < 1) slices = 1;
    const int waves = KQ <= 16 ? KQ * slices : 16;
    const int lds_slices = waves >= KQ ? waves / KQ : 1;
    // int F[N] | int n | 1 pad int  keeps the Best array that follows 16-byte aligned when N is even; round up
    size_t lds = sizeof(double) * (static_cast<size_t>(S < 0 ? N : N - S) * KP + K + N) + sizeof(int) * (static_cast<size_t>(N) + 3);
    lds += 16 + sizeof(double) * 2 * static_cast<size_t>(KP) * lds_slices;
    const dim3 grid(static_cast<unsigned>(G)), block(waves * kWave);
    if (lds > 64 * 1024) {
        const void *fn = vec4 ? reinterpret_cast<const void *>(decode_top1_kernel<4>)
                              : reinterpret_cast<const void *>(decode_top1_kernel<1>);
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
            return APPROXIFER_ERR_LAUNCH;
    }
    return launch_status(launch_kernel(vec4 ? decode_top1_kernel<4> : decode_top1_kernel<1>, grid, block, lds, stream,
                                       d_preds, d_mask, d_top1, d_score, d_status, K, N, S, C, Cv, sign_mode, nodes));
}

int launch_argmax_rows(const float *d_values, int32_t *d_top1, float *d_score, int64_t rows, int64_t C,
                       hipStream_t stream) {
    const bool narrow = C <= 32;
    const int64_t per_block = kArgmaxWaves * (narrow ? kWave / 16 : 1);
    const int64_t blocks = (rows + per_block - 1) / per_block;
    if (blocks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const dim3 grid(static_cast<unsigned>(blocks)), block(kArgmaxWaves * kWave);
    if (narrow) return launch_status(launch_kernel(argmax_rows_kernel<16>, grid, block, 0, stream, d_values, d_top1, d_score, rows, C));
    return launch_status(launch_kernel(argmax_rows_kernel<kWave>, grid, block, 0, stream, d_values, d_top1, d_score, rows, C));
}

int launch_wait_mask(const float *d_arrival, uint8_t *d_mask, int32_t *d_count, int64_t G, int N, int wait_for,
                     hipStream_t stream) {
    const int64_t blocks = (G + kWaitGroups - 1) / kWaitGroups;
    if (blocks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    return launch_status(launch_kernel(wait_mask_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kWaitGroups * kWave), 0,
                                       stream, d_arrival, d_mask, d_count, G, N, wait_for));
}

}  // namespace approxifer

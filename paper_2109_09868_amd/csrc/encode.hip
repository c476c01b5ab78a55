// ApproxIFER encoder for gfx950 (Section 3, "ApproxIFER Encoding").
//
//   coded[g][i][d] = sum_j l_j(beta_i) * queries[g][j][d]
//
// One workgroup per (group, tile of vector columns): a single wave (64 columns) for K <= 16 and rows of 16-byte
// pieces, four waves (256 columns) otherwise; rows that leave lanes idle at their end are tiled over the
// flattened (group, column) index instead, and rows that are not whole 64-byte sectors go by tiles whose stores are
// (encode_sectors_kernel, encode_mfma_sectors_kernel) where that is the faster side (sector_rows).  Each lane first issues the loads of its vector column of
// all K queries (they stay in registers), and while those are in flight the workgroup
// evaluates the N x K matrix l_j(beta_i) -- it depends on the nodes only -- in float64 (one
// 16/32/64-lane group per worker row, the row's denominator by a DPP reduction) and keeps it
// in LDS as float32.  The N coded values of the column are then formed one worker at a time
// with the weights broadcast from LDS and stored as soon as complete.
// Every query element is read from HBM exactly once and every coded element written exactly
// once: the kernel is an HBM stream of 4*D*(K+N) bytes per group with 2*K*N flops per
// 4*(K+N) bytes on top.
//
// Two launch-shape facts, both measured on MI355X at the 3x224x224, K=12, N=20 shape:
//  * Workgroups do not loop over tiles.  On gfx9 one counter orders a wave's loads and stores,
//    so a looping wave waits for its previous stores before it can use its next loads; a wave
//    that retires after issuing its stores does not (1.92 ms persistent, 1.76 ms one-shot).
//  * HBM efficiency falls with the number of row streams that are open at once (a plain copy
//    reaches 6.6 TB/s walked sequentially, 5.2 TB/s walked as 12+12 interleaved rows), i.e.
//    with the number of tiles in flight.  The kernel therefore caps residency at a few waves
//    per CU by reserving LDS it does not use: each wave has all K of its 128-bit loads in flight,
//    which is enough to cover latency (1.76 ms uncapped, 1.60 ms at 6 waves per CU).
#include "common.h"
#include "sectors.h"

namespace approxifer {
namespace {

// Residency caps (workgroups per CU), from sweeps on the benchmark shapes and on a K x N x D grid.
// K <= 16, one-wave workgroups: enough waves to keep about 48 KB of query loads in flight per CU (a wave
// has K loads of 1 KB each), never fewer than six and never more than 24: measured optima are 20+ at K = 1,
// 12..16 at K = 2, 8..12 at K = 4..6, 6 at K = 8..16 (7 and up lose 1..4 % there: more row streams open).
constexpr int kWavesPerCuMin = 6;
constexpr int kLoadKbPerCu = 48;
constexpr int kBlocksPerCuLargeK = 2;   // K > 16: four-wave workgroups
constexpr int kMfmaMinK = 17;   // from this K on the matrix-core variant serves every shape
constexpr int kMfmaWideMinK = 8;   // .. and from this K on the shapes with N >= 2K + 4
constexpr int kMfmaBlocksPerCu = 4;   // matrix-core variant (four waves of 64 columns)
constexpr int kSectorRowsMinD = 129;   // rows that are not whole 64-byte sectors: tiles of whole sectors from here on
constexpr int kSectorMinTiles = 2048;   // .. if rows are 16-byte pieces, for calls of this many tiles or more
constexpr int kSectorFewTiles = 640;   // calls whose time is the chain of one workgroup (see sector_rows)
constexpr int kMfmaSectorsMinD = 300;   // K <= 16: .. on the matrix cores, where they pay, from here on; shorter rows: see sector_rows
constexpr int kScalarRowsMaxD = 128;   // ragged rows (D % 4 != 0) this short: 64-bit or 4-byte accesses only

// Register type of VEC floats, and the type a lane loads and stores it through.  Rows that are only
// 4-byte aligned (a row length that is not a multiple of 4 floats, or an offset base pointer) are still
// moved 128 bits at a time: gfx950 serves dword-aligned 128-bit global accesses, and the compiler emits them
// for a vector type declared with 4-byte alignment.
template <int VEC> struct VecOf;
template <> struct VecOf<4> { typedef v4f type; };
template <> struct VecOf<2> { typedef v2f type; };
template <> struct VecOf<1> { typedef float type; };
typedef v4f v4f_align4 __attribute__((aligned(4)));
template <int VEC, bool UNAL> struct MemOf { typedef typename VecOf<VEC>::type type; };
template <> struct MemOf<4, true> { typedef v4f_align4 type; };

template <int VEC, bool UNAL = false>
__device__ __forceinline__ typename VecOf<VEC>::type load_stream(const float *p) {
    typedef typename MemOf<VEC, UNAL>::type M;
    const M v = __builtin_nontemporal_load(reinterpret_cast<const M *>(p));
    return v;
}
template <int VEC, bool UNAL = false>
__device__ __forceinline__ void store_stream(float *p, typename VecOf<VEC>::type v) {
    typedef typename MemOf<VEC, UNAL>::type M;
    __builtin_nontemporal_store(static_cast<M>(v), reinterpret_cast<M *>(p));
}

// ---- l_j(beta_i) in float64, one group of LPR lanes per worker row ---------------------
// The nodes are read with compile-time or wave-uniform indices only, i.e. through scalar
// loads: a vector load here would queue behind the query loads above and make the wave
// wait for all of them before it could evaluate a single weight.
template <int K, int THREADS>
__device__ __forceinline__ void encode_weights(float *wl, int N, const Nodes &nodes) {   // wl[N][KP]
    constexpr int KP = (K + 3) & ~3;       // weight row padded to whole float4s
    constexpr int LPR = K <= 16 ? 16 : (K <= 32 ? 32 : 64);   // lanes per weight row
    constexpr int ROWS_PER_PASS = THREADS / LPR;
    const int tid = threadIdx.x;
    const int j = tid % LPR;
    const int sub = tid / LPR;
    const bool valid = j < K;
    double xa = 0.0;
#pragma unroll
    for (int jj = 0; jj < K; ++jj) {
        const double a = wave_uniform(nodes.alpha[jj]);
        if (j == jj) xa = a;
    }
    const double sign = (j & 1) ? -1.0 : 1.0;
    for (int i0 = 0; i0 < N; i0 += ROWS_PER_PASS) {   // i0 + ROWS_PER_PASS <= APPROXIFER_MAX_N always
        double z = wave_uniform(nodes.beta[i0]);
#pragma unroll
        for (int r = 1; r < ROWS_PER_PASS; ++r) {
            const double zr = wave_uniform(nodes.beta[i0 + r]);
            if (sub == r) z = zr;
        }
        const int i = i0 + sub;
        const bool row = i < N;
        const BerrutTerm bt = berrut_term(z, xa, sign, valid && row);
        const double den = group_sum<LPR>(bt.t);
        const unsigned long long hits = __ballot(bt.hit);
        const unsigned long long group_mask = (LPR == 64) ? ~0ull : ((1ull << (LPR & 63)) - 1ull) << ((tid & 63) / LPR * LPR);
        const bool any_hit = (hits & group_mask) != 0ull;
        const double w = any_hit ? (bt.hit ? 1.0 : 0.0) : bt.t * (1.0 / den);
        if (row && j < KP) wl[i * KP + j] = valid ? static_cast<float>(w) : 0.0f;
    }
}

// K: queries per group (compile time so that the K input columns stay in registers).
// VEC: floats per lane per access.  THREADS: workgroup size.
// FLAT: false -- a workgroup covers THREADS consecutive vector columns of ONE group (`chunks` workgroups per
//       group; the last one of a group may be partly idle);  true -- the (group, vector column) pairs of the
//       whole batch are numbered consecutively and a workgroup takes THREADS of them, so lanes never idle at a
//       row end.  Used when rows are short and ragged (28 x 28 queries: 196 vector columns, 23 % idle lanes
//       otherwise); `chunks` then carries the total number of pairs.
// UNAL: rows are only 4-byte aligned (VEC == 4 accesses then go through the 4-byte-aligned vector type).
// col0: first float column served; columns col0 + VEC * [0, Dv) are produced.
template <int K, int VEC, int THREADS, bool FLAT, bool UNAL>
__global__ __launch_bounds__(THREADS) void encode_kernel(
    const float *__restrict__ queries, float *__restrict__ coded, int N, int64_t D, int64_t Dv,
    int64_t chunks, int64_t col0, const Nodes nodes) {
    typedef typename VecOf<VEC>::type V;
    constexpr int KP = (K + 3) & ~3;
    extern __shared__ float wl[];          // [N][KP]

    const int tid = threadIdx.x;
    int64_t g, col;
    bool ok;
    if (FLAT) {
        const int64_t q = static_cast<int64_t>(blockIdx.x) * THREADS + tid;
        ok = q < chunks;
        const int64_t qq = ok ? q : 0;
        if (chunks <= 0xffffffffLL) {      // the usual case: one 32-bit division per lane
            const uint32_t g32 = static_cast<uint32_t>(qq) / static_cast<uint32_t>(Dv);
            g = g32;
            col = static_cast<uint32_t>(qq) - g32 * static_cast<uint32_t>(Dv);
        } else {
            g = qq / Dv;
            col = qq - g * Dv;
        }
    } else {
        g = blockIdx.x / chunks;
        col = (blockIdx.x - g * chunks) * THREADS + tid;
        ok = col < Dv;
        if (!ok) col = 0;                  // lanes past the ragged end read column 0 of the group and store nothing
    }
    const float *xg = queries + static_cast<size_t>(g) * K * D + col0 + col * VEC;
    float *og = coded + static_cast<size_t>(g) * N * D + col0 + col * VEC;

    // ---- this lane's column of the K queries: issue every load before anything else ----
    V x[K];
#pragma unroll
    for (int j = 0; j < K; ++j) x[j] = load_stream<VEC, UNAL>(xg + static_cast<size_t>(j) * D);

    encode_weights<K, THREADS>(wl, N, nodes);
    __syncthreads();

    const v4f *wl4 = reinterpret_cast<const v4f *>(wl);
    for (int i = 0; i < N; ++i) {
        V acc = V(0.0f);
#pragma unroll
        for (int j4 = 0; j4 < KP / 4; ++j4) {
            const v4f w = wl4[i * (KP / 4) + j4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                if (4 * j4 + jj < K) acc = w[jj] * x[4 * j4 + jj] + acc;
        }
        if (ok) store_stream<VEC, UNAL>(og + static_cast<size_t>(i) * D, acc);
    }
}

// The same on tiles of whole sectors (see store_sectors): a tile per wave, K <= 16.  An HBM stream as above; what the
// unaligned stores cost it was a fifth (K = 8, N = 12, 64 groups of 3 x 299 x 299 floats: 270 -> 231 us, 5.1 -> 5.9 TB/s; rows of
// 268288 floats, all sectors whole: 218 us).  Four waves to a workgroup, so that three of four halos are read through one L2:
// with a wave each 250 us.
template <int K, int THREADS>
__global__ __launch_bounds__(THREADS) void encode_sectors_kernel(
    const float *__restrict__ queries, float *__restrict__ coded, int N, int64_t D, uint32_t per_row, int width,
    uint32_t tiles, const Nodes nodes) {
    extern __shared__ float wl[];          // [N][KP]
    constexpr int KP = (K + 3) & ~3;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const uint32_t id = blockIdx.x * (THREADS / kWave) + __builtin_amdgcn_readfirstlane(wave_id());
    const RowTile t = row_tile(id < tiles ? id : 0, per_row, width, kTileHalo, D);
    const int c = t.column(lane);
    const float *xg = queries + static_cast<size_t>(t.g) * K * D + load_column(t, c, D);

    v4f x[K];
#pragma unroll
    for (int j = 0; j < K; ++j) x[j] = load_stream<4, true>(xg + static_cast<size_t>(j) * D);
    encode_weights<K, THREADS>(wl, N, nodes);
    __syncthreads();
    if (id >= tiles) return;               // no barrier left

    if (t.last && D % 4 != 0) {
        const bool over = over_the_end(t, c);
#pragma unroll
        for (int j = 0; j < K; ++j) x[j] = finish_vector(x[j], over, static_cast<int>(D % 4));
    }
    float *row = coded + static_cast<size_t>(t.g) * N * D + t.start;
    int at = static_cast<int>(reinterpret_cast<uintptr_t>(row) / sizeof(float)) & (kSector - 1);
    const v4f *wl4 = reinterpret_cast<const v4f *>(wl);
    for (int i = 0; i < N; ++i) {
        v4f acc = v4f(0.0f);
#pragma unroll
        for (int j4 = 0; j4 < KP / 4; ++j4) {
            const v4f w = wl4[i * (KP / 4) + j4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                if (4 * j4 + jj < K) acc = w[jj] * x[4 * j4 + jj] + acc;
        }
        store_sectors(row, acc, c, at, t);
        row += D;
        at = (at + static_cast<int>(D & (kSector - 1))) & (kSector - 1);
    }
}

// ---- matrix-core variant for K > 16 -----------------------------------------------------
// At K = 32, N = 48 the vector kernel above issues VALU instructions on 95 % of all cycles
// (SQ_INSTS_VALU x 4 against SIMD-cycles): the contraction, not HBM, bounds it there.  This
// variant forms coded = W (N x K) * X (K x columns) with v_mfma_f32_16x16x4_f32, whose fp32 rate is
// twice the plain vector FMA rate, and leaves the vector ALUs to address arithmetic.
//
// Operand layout of v_mfma_f32_16x16x4_f32 (D[16x16] += A[16x4] * B[4x16]), lane l of the wave:
//   A: element (row l%16, k l/16)       B: element (k l/16, column l%16)
//   D: register r holds element (row 4*(l/16) + r, column l%16)
// A wave owns 64 consecutive columns of a group.  One 128-bit load gives lane l the four columns
// 4*(l%16)..+3 of query row 4s + l/16, so component e of that register IS the B operand of k-step
// s for the column set {4c + e}: no shuffles.  The four column sets give, in register r of their
// accumulators, four consecutive columns of worker row 16*mt + 4*(l/16) + r: one 128-bit store.
// The weights sit in LDS already in A-operand order, wA[(mt*KS + s)*64 + l].
constexpr int kMfmaThreads = 256;

// l_j(beta_i) in float64 (scalar node loads only, see encode_weights), stored in A order
template <int KS>
__device__ __forceinline__ void encode_mfma_weights(float *wA, int K, int N, const Nodes &nodes) {
    constexpr int LPR = KS <= 8 ? 32 : 64;                    // lanes per weight row (K <= 32 / K <= 64)
    constexpr int ROWS_PER_PASS = kMfmaThreads / LPR;
    const int tid = threadIdx.x;
    const int j = tid % LPR;
    const int sub = tid / LPR;
    const bool valid = j < K;
    double xa = 0.0;
#pragma unroll
    for (int jj = 0; jj < 4 * KS; ++jj) {
        const double a = wave_uniform(nodes.alpha[jj]);   // entries past K are zero-filled by the host
        if (j == jj) xa = a;
    }
    const double sign = (j & 1) ? -1.0 : 1.0;
    const int n16 = (N + 15) & ~15;
    for (int i0 = 0; i0 < n16; i0 += ROWS_PER_PASS) {     // n16 <= 128 = APPROXIFER_MAX_N: reads stay in bounds
        double z = wave_uniform(nodes.beta[i0]);
#pragma unroll
        for (int r = 1; r < ROWS_PER_PASS; ++r) {
            const double zr = wave_uniform(nodes.beta[i0 + r]);
            if (sub == r) z = zr;
        }
        const int i = i0 + sub;
        const bool row = i < N;
        const BerrutTerm bt = berrut_term(z, xa, sign, valid && row);
        const double den = group_sum<LPR>(bt.t);
        const unsigned long long hits = __ballot(bt.hit);
        const unsigned long long group_mask =
            (LPR == 64) ? ~0ull : ((1ull << (LPR & 63)) - 1ull) << ((tid & 63) / LPR * LPR);
        const bool any_hit = (hits & group_mask) != 0ull;
        const double w = any_hit ? (bt.hit ? 1.0 : 0.0) : bt.t * (1.0 / den);
        if (j < 4 * KS)   // rows N..n16-1 and columns K..4KS-1 hold zeros
            wA[((i >> 4) * KS + (j >> 2)) * 64 + (j & 3) * 16 + (i & 15)] = (valid && row) ? static_cast<float>(w) : 0.0f;
    }
}

// KS = ceil(K / 4) k-steps; UNAL: rows only 4-byte aligned; FLAT: the 16-column wave tiles run over the flattened
// (group, vector column) numbering of the batch (`chunks` = number of pairs), as in encode_kernel.
template <int KS, bool UNAL, bool FLAT>
__global__ __launch_bounds__(kMfmaThreads) void encode_mfma_kernel(
    const float *__restrict__ queries, float *__restrict__ coded, int K, int N, int64_t D, int64_t Dv,
    int64_t chunks, const Nodes nodes) {
    extern __shared__ float wA[];                             // [ceil(N/16)][KS][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = tid >> 6;
    int64_t g, col;                                           // this lane's group and vector column
    bool ok;
    if (FLAT) {
        const int64_t q = (static_cast<int64_t>(blockIdx.x) * (kMfmaThreads / 64) + wv) * 16 + (lane & 15);
        ok = q < chunks;
        const int64_t qq = ok ? q : 0;
        if (chunks <= 0xffffffffLL) {
            const uint32_t g32 = static_cast<uint32_t>(qq) / static_cast<uint32_t>(Dv);
            g = g32;
            col = static_cast<uint32_t>(qq) - g32 * static_cast<uint32_t>(Dv);
        } else {
            g = qq / Dv;
            col = qq - g * Dv;
        }
    } else {
        g = blockIdx.x / chunks;
        col = ((blockIdx.x - g * chunks) * (kMfmaThreads / 64) + wv) * 16 + (lane & 15);
        ok = col < Dv;
        if (!ok) col = 0;
    }
    const int krow = lane >> 4;                               // row offset inside a k-step
    // a row's last, partial vector is loaded as the last four floats of the row and shifted down below (a launch of its own for the
    // last columns costs its weights again: K = 40, N = 88, four rows of 73 floats 29.5 and 18.3 us)
    const int tail = UNAL ? static_cast<int>(D & 3) : 0;
    const bool over = tail != 0 && col == Dv - 1;
    const float *xg = queries + static_cast<size_t>(g) * K * D + (over ? D - 4 : col * 4);
    float *og = coded + static_cast<size_t>(g) * N * D + col * 4;

    // ---- query rows 4s + krow, columns 4*col..+3; rows past K (KS = ceil(K / 4)) are clamped, and zeroed below ----
    v4f x[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int row = (4 * s + krow < K) ? 4 * s + krow : K - 1;
        x[s] = load_stream<4, UNAL>(xg + static_cast<size_t>(row) * D);
    }

    encode_mfma_weights<KS>(wA, K, N, nodes);
    __syncthreads();
    if (UNAL && tail != 0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = finish_vector(x[s], over, tail);
    }
    if (4 * (KS - 1) + krow >= K) x[KS - 1] = v4f(0.0f);      // a clamped row: its infinities count for nothing either

    const int mtiles = (N + 15) >> 4;
    for (int mt = 0; mt < mtiles; ++mt) {
        v4f acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = v4f(0.0f);
        const float *wmt = wA + mt * KS * 64 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float a = wmt[s * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, x[s][e], acc[e], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * mt + 4 * krow + r;
            if (ok && i < N) {
                v4f v;
                v[0] = acc[0][r];
                v[1] = acc[1][r];
                v[2] = acc[2][r];
                v[3] = acc[3][r];
                float *row = og + static_cast<size_t>(i) * D;
                if (!UNAL || !over) {
                    store_stream<4, UNAL>(row, v);
                } else {
                    row[0] = v[0];
                    if (tail > 1) row[1] = v[1];
                    if (tail > 2) row[2] = v[2];
                }
            }
        }
    }
}

// The same on tiles of whole sectors (see store_sectors), one tile of 64 vectors per workgroup: the waves compute sixteen
// vectors each, as above, and exchange the sixteen coded rows of a round through LDS, from where each wave stores
// four rows as they lie in memory.  (A wave's own sixteen vectors end inside a sector on both sides: five pieces for four.)
// An HBM stream: K = 32, N = 48, 93 groups of 10003 floats 100 -> 65 us (4.6 TB/s; a quarter more is read than the queries hold);
// K = 12, N = 28, 187 groups 87 -> 57 us (5.3 TB/s).  Launch after launch; the first on new buffers 74 and 68.
// dynamic LDS: float wA[ceil(N/16)][KS][64] | stage[16][kStageRow]
constexpr int kStageRow = 256 + 4;
template <int KS>
__global__ __launch_bounds__(kMfmaThreads) void encode_mfma_sectors_kernel(
    const float *__restrict__ queries, float *__restrict__ coded, int K, int N, int64_t D, uint32_t per_row, int width,
    const Nodes nodes) {
    extern __shared__ __align__(16) float wA[];
    const int mtiles = (N + 15) >> 4;
    float *stage = wA + mtiles * KS * 64;
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());
    const RowTile t = row_tile(blockIdx.x, per_row, width, kTileHalo, D);
    const int krow = lane >> 4;
    const int vec = wv * 16 + (lane & 15);                    // this lane's vector of the tile while computing
    const int c = t.column(vec);
    const float *xg = queries + static_cast<size_t>(t.g) * K * D + load_column(t, c, D);
    v4f x[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int row = (4 * s + krow < K) ? 4 * s + krow : K - 1;
        x[s] = load_stream<4, true>(xg + static_cast<size_t>(row) * D);
    }
    encode_mfma_weights<KS>(wA, K, N, nodes);
    __syncthreads();
    if (t.last && D % 4 != 0) {
        const bool over = over_the_end(t, c);
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = finish_vector(x[s], over, static_cast<int>(D % 4));
    }
    if (4 * (KS - 1) + krow >= K) x[KS - 1] = v4f(0.0f);      // a clamped row, see encode_mfma_kernel

    float *og = coded + static_cast<size_t>(t.g) * N * D + t.start;
    for (int mt = 0; mt < mtiles; ++mt) {
        v4f acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = v4f(0.0f);
        const float *wmt = wA + mt * KS * 64 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float a = wmt[s * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, x[s][e], acc[e], 0, 0, 0);
        }
        if (mt > 0) __syncthreads();                          // the rows of the round before are stored
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<v4f *>(stage + (4 * krow + r) * kStageRow + 4 * vec) = v4f{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * mt + 4 * wv + r;
            if (i < N) {
                float *row = og + static_cast<size_t>(i) * D;
                const int at = static_cast<int>(reinterpret_cast<uintptr_t>(row) / sizeof(float)) & (kSector - 1);
                store_sectors(row, *reinterpret_cast<const v4f *>(stage + (4 * wv + r) * kStageRow + 4 * lane), t.column(lane), at, t);
            }
        }
    }
}

template <int KS, bool UNAL, bool FLAT>
int run_encode_mfma_shape(const float *d_queries, float *d_coded, int64_t tiles, int64_t chunks, int K, int N, int64_t D,
                          int64_t Dv, const Nodes &nodes, hipStream_t stream) {
    if (tiles > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const size_t lds_used = static_cast<size_t>((N + 15) / 16) * KS * 64 * sizeof(float);
    size_t lds = (static_cast<size_t>(kLdsPerCu / kMfmaBlocksPerCu) / 512) * 512;
    if (lds < lds_used) lds = lds_used;
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(encode_mfma_kernel<KS, UNAL, FLAT>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(encode_mfma_kernel<KS, UNAL, FLAT>, dim3(static_cast<unsigned>(tiles)),
                                       dim3(kMfmaThreads), lds, stream, d_queries, d_coded, K, N, D, Dv, chunks, nodes));
}

template <int KS, bool UNAL>
int run_encode_mfma(const float *d_queries, float *d_coded, int64_t G, int K, int N, int64_t D, const Nodes &nodes,
                    hipStream_t stream) {
    const int64_t Dv = UNAL ? (D + 3) / 4 : D / 4;                      // counts a partial last vector
    const int64_t cols_per_block = (kMfmaThreads / 64) * 16;           // vector columns per workgroup
    const int64_t chunks = (Dv + cols_per_block - 1) / cols_per_block;
    const int64_t idle = chunks * cols_per_block - Dv;                  // columns without data at the row ends
    const int64_t pairs = G * Dv;
    const int64_t flat = (pairs + cols_per_block - 1) / cols_per_block;
    if constexpr (!UNAL)                                                // UNAL: short rows, or few (sector_rows)
        if (idle * 100 <= 3 * chunks * cols_per_block)
            return run_encode_mfma_shape<KS, false, false>(d_queries, d_coded, G * chunks, chunks, K, N, D, Dv, nodes, stream);
    return run_encode_mfma_shape<KS, UNAL, true>(d_queries, d_coded, flat, pairs, K, N, D, Dv, nodes, stream);
}

// Workgroup size.  K <= 16: one wave, but four for rows that are only 4-byte aligned (short ones, or few: the others go by tiles
// of whole sectors).
constexpr int encode_threads(int K, bool UNAL) { return K <= 16 && !UNAL ? 64 : 256; }

// Workgroups per CU, where the stage and the weights leave room for them (six, eight and four at 300 MB: K = 12, N = 28,
// 350 floats 76, 73, 79 us, 10003 floats 56, 58, 58; K = 8, N = 24, 350 floats 81, 75, 88, 10003 floats 57, 58, 60; with two
// stages, a barrier less, and four 58 to 61 at 10003 floats).
constexpr int mfma_sector_blocks(int64_t D) { return D < 2048 ? 8 : 6; }

template <int KS>
int run_encode_mfma_sectors(const float *d_queries, float *d_coded, int64_t G, int K, int N, int64_t D, const Nodes &nodes,
                            hipStream_t stream) {
    const SectorTiles t = sector_tiles(G, D, kTileHalo);
    if (t.total > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const size_t lds_used = (static_cast<size_t>((N + 15) / 16) * KS * 64 + 16 * kStageRow) * sizeof(float);
    size_t lds = (static_cast<size_t>(kLdsPerCu / mfma_sector_blocks(D)) / 512) * 512;
    if (lds < lds_used) lds = lds_used;
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(encode_mfma_sectors_kernel<KS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(encode_mfma_sectors_kernel<KS>, dim3(static_cast<unsigned>(t.total)), dim3(kMfmaThreads),
                                       lds, stream, d_queries, d_coded, K, N, D, static_cast<uint32_t>(t.per_row), t.width,
                                       nodes));
}

// Workgroups of four waves per CU: with K <= 4 loads a wave, or rows of a few tiles that leave lanes idle, sixteen waves keep
// enough bytes in flight; from five loads and 8 KB a row on, eight.  16 and 8 waves at N = K + 1 .. 1.5 K, 300 MB: K = 4, 1425
// floats 52 and 59 us, 50001 floats 49 and 53; K = 8, 477 floats 66 and 80, 604 floats 58 and 59, 3075 floats 58 and 56.  Calls
// of up to 4096 tiles have sixteen, which is all of them at once, up to twelve queries (2049 tiles and more: K = 5 and 6 0.885 of
// the time, 11 and 12 0.95, 15 and 16 0.99), and hardly more than one round of sixteen, up to 4800 tiles, are one of twenty-four (0.92 to
// 0.98; beyond eight queries 1.02 where eight waves are the usual).
constexpr int sector_blocks(int K, int64_t D, int64_t tiles) {
    if (K <= 2) return 6;
    const int usual = K <= 4 || D < 2048 ? 4 : 2;
    if (tiles <= 4096) return K <= 12 ? 4 : usual;
    return tiles <= 4800 && (usual == 4 || K <= 8) ? 6 : usual;
}

template <int K>
int run_encode_sectors(const float *d_queries, float *d_coded, int64_t G, int N, int64_t D, const Nodes &nodes,
                       hipStream_t stream) {
    constexpr int KP = (K + 3) & ~3;
    constexpr int THREADS = 256;
    const SectorTiles t = sector_tiles(G, D, kTileHalo);
    if (t.total > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const int per_cu = sector_blocks(K, D, t.total);
    const size_t lds_used = static_cast<size_t>(N) * KP * sizeof(float);
    size_t lds = (static_cast<size_t>(kLdsPerCu / per_cu) / 512) * 512;
    if (lds < lds_used) lds = lds_used;
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(encode_sectors_kernel<K, THREADS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(encode_sectors_kernel<K, THREADS>,
                                       dim3(static_cast<unsigned>((t.total + THREADS / 64 - 1) / (THREADS / 64))), dim3(THREADS),
                                       lds, stream, d_queries, d_coded, N, D, static_cast<uint32_t>(t.per_row), t.width,
                                       static_cast<uint32_t>(t.total), nodes));
}

template <int K, int VEC, bool FLAT, bool UNAL>
int run_encode_shape(const float *d_queries, float *d_coded, int64_t tiles, int64_t chunks, int N, int64_t D,
                     int64_t Dv, int64_t col0, const Nodes &nodes, hipStream_t stream) {
    constexpr int KP = (K + 3) & ~3;
    constexpr int THREADS = encode_threads(K, UNAL);
    int per_cu = kBlocksPerCuLargeK;
    if (K <= 16) {
        per_cu = (kLoadKbPerCu + K - 1) / K;     // K loads of 1 KB per wave
        if (per_cu < kWavesPerCuMin) per_cu = kWavesPerCuMin;
        if (per_cu > 24) per_cu = 24;
        if (THREADS > 64) per_cu = (per_cu + THREADS / 64 - 1) / (THREADS / 64);   // as many waves, up to whole workgroups
        if (VEC == 1) per_cu = 7;       // 4-byte accesses: ragged rows of up to 128 floats, or the last D % 4 columns
    }
    if (tiles > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    const size_t lds_used = static_cast<size_t>(N) * KP * sizeof(float);
    // reserve 1/per_cu of the CU's LDS so that at most per_cu workgroups are resident
    size_t lds = (static_cast<size_t>(kLdsPerCu / per_cu) / 512) * 512;
    if (lds < lds_used) lds = lds_used;
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(encode_kernel<K, VEC, THREADS, FLAT, UNAL>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return APPROXIFER_ERR_LAUNCH;
    return launch_status(launch_kernel(encode_kernel<K, VEC, THREADS, FLAT, UNAL>, dim3(static_cast<unsigned>(tiles)),
                                       dim3(THREADS), lds, stream, d_queries, d_coded, N, D, Dv, chunks, col0, nodes));
}

// Vector columns [0, Dv) of width VEC floats, starting at float column col0.
template <int K, int VEC, bool UNAL>
int run_encode(const float *d_queries, float *d_coded, int64_t G, int N, int64_t D, int64_t Dv, int64_t col0,
               const Nodes &nodes, hipStream_t stream) {
    constexpr int THREADS = encode_threads(K, UNAL);
    const int64_t chunks = (Dv + THREADS - 1) / THREADS;
    // lanes left idle at the row ends by the per-group tiling; above 3 % the flattened numbering pays for its
    // per-lane division and addresses
    const int64_t idle = chunks * THREADS - Dv;
    const int64_t pairs = G * Dv;
    const int64_t flat = (pairs + THREADS - 1) / THREADS;
    if constexpr (!UNAL)                                      // UNAL: short rows, or few (sector_rows)
        if (idle * 100 <= 3 * chunks * THREADS)
            return run_encode_shape<K, VEC, false, false>(d_queries, d_coded, G * chunks, chunks, N, D, Dv, col0, nodes, stream);
    return run_encode_shape<K, VEC, true, UNAL>(d_queries, d_coded, flat, pairs, N, D, Dv, col0, nodes, stream);
}

// 16-byte-aligned rows: the matrix-core kernel or the vector kernel, by shape.
template <int K>
int run_encode_wide(const float *d_queries, float *d_coded, int64_t G, int N, int64_t D, const Nodes &nodes,
                    hipStream_t stream) {
    if constexpr (K >= kMfmaMinK) {
        return run_encode_mfma<(K + 3) / 4, false>(d_queries, d_coded, G, K, N, D, nodes, stream);
    } else {
        if constexpr (K >= kMfmaWideMinK) {
            // Many more coded than plain queries (the Byzantine worker counts, N = 2 (K + A) + S): a one-wave
            // tile would keep K + N >= 3K + 4 row streams open, and the matrix-core variant, whose waves work on
            // 256-byte row segments, measures 4..14 % faster (K=8, N=24: 5.7 -> 6.2 TB/s; K=12, N=36: 5.5 -> 6.0).
            if (N >= 2 * K + 4)
                return run_encode_mfma<(K + 3) / 4, false>(d_queries, d_coded, G, K, N, D, nodes, stream);
        }
        return run_encode<K, 4, false>(d_queries, d_coded, G, N, D, D / 4, 0, nodes, stream);
    }
}

// Whether a call goes by tiles of whole sectors: rows that are no whole sectors, of kSectorRowsMinD floats or more.  Both sides
// timed over 5000 calls of 1 to 64 queries, 129 to 280000 floats, up to 1.2 GB; times without and with the tiles.
//  - Rows that are only 4-byte aligned: nearly all calls gain (0.78 of the time on average; K = 8, N = 12, 64 x 3 x 299 x 299 floats 270
//    and 231 us; K = 32, N = 48, 93 x 10003 100 and 65).  Not K = 20, N = 24 with tiles of fewer than forty own vectors (156
//    floats 74 and 78 us, 258 floats 86 and 98); not K < 8 with sixteen or more workers in few short rows, whose time is one
//    wave's chain of coded rows (K = 4, N = 16, 19 groups of 141 floats 7.6 and 8.7 us); not many small groups of a single query
//    (12642 of 275 floats, N = 2 13.3 and 15.3).
//  - Rows of 16-byte pieces lose only the sectors at the ends of a wave's segment, and only where HBM takes them:
//    K > 32: none (K = 39, N = 54, 128 x 8132 floats 90 and 100 us; 1.05 times at K = 36, 1.2 times at K = 64).  K = 17..32: from 2048
//    tiles on, rows of one tile of 45 vectors and more (K = 26, N = 31, 196 floats 166 and 127 us); tiles of more than forty own
//    vectors where the coded rows are many (N >= 2 K: 0.82 of the time), of more than fifty from 1.5 K on (0.92), and with fewer
//    yet of more than 54 and not for D % 8 = 0, which cuts fewer sectors (0.92; K = 17, N = 18, 20000 tiles of 1004 floats 132 and
//    155 us).  K <= 16: calls of 8 MB a query and more (64 MB from eight on, and for K = 1), half that where N >= 2 K + 4, else twice
//    that in tiles of fewer than fifty own vectors: 0.90 of the time above, 1.01 below (K = 4, N = 6, 2692 x 260 floats 7.4 and 8.9
//    us; K = 6, N = 12, 193 x 2700 floats 9.4 and 10.9; K = 1, N = 9, 4 x 153684 floats 7.9 and 5.8).  Not rows of 63
//    vectors, which are one wave each as they come (252 floats: 1.0 to 1.17 times), nor many small tiles of a single query with two
//    workers (8702 x 1484 floats 28.8 and 30.4), nor rows of whole 32-byte pieces (D % 8 = 0), which cut half as many sectors, in little
//    more than one round of workgroups (three to five queries, N < 2 K; K = 3, N = 5, 1296 x 792 floats 7.5 and 8.9).  From eight queries and N = 2 K + 4 on they
//    stand against the matrix-core kernel: on the matrix cores in tiles of 48 vectors and more (K = 16, N = 40, 758 x 504 floats
//    22 and 28 us), and for rows of one tile of up to 56 vectors (K = 14, N = 35, 11377 x 156 floats 114 and 88 us; K = 8, N = 23,
//    9020 x 252 floats 53 and 67), of whole 32-byte pieces only on the matrix cores and from 23 workers on (K = 14, N = 35, 4352 x 136
//    floats 1.10 times; K = 8, N = 20, 1588 x 776 30.4 and 35.4; N = 23..28 0.87 to 0.99).
inline bool sector_rows(const float *d_queries, const float *d_coded, int64_t G, int K, int N, int64_t D) {
    if ((whole_sectors(d_queries, D) && whole_sectors(d_coded, D)) || D < kSectorRowsMinD) return false;
    const bool pieces = D % 4 == 0 && reinterpret_cast<uintptr_t>(d_queries) % 16 == 0 && reinterpret_cast<uintptr_t>(d_coded) % 16 == 0;
    const SectorTiles t = sector_tiles(G, D, kTileHalo);
    const int own = t.width / 4;
    if (!pieces) {
        if (K >= kMfmaMinK) return 2 * N >= 3 * K || own >= 40;
        if (K == 1 && N <= 4 && own < 44 && t.total >= 8192) return false;
        return K >= kMfmaWideMinK || N < 16 || D >= kMfmaSectorsMinD || t.total > kSectorFewTiles;
    }
    if (K >= kMfmaMinK) {
        if (K > 32 || t.total < kSectorMinTiles) return false;
        if (t.per_row == 1) return own >= 45;
        return N >= 2 * K ? own > 40 : (2 * N >= 3 * K ? own > 50 : own > 54 && D % 8 != 0);
    }
    const bool many = N >= 2 * K + 4, half = D % 8 == 0;
    if (t.per_row == 1 && own == 63) return false;
    if (K >= kMfmaWideMinK && many) {
        if (half && (N <= 22 || D < kMfmaSectorsMinD)) return false;
        if (D < kMfmaSectorsMinD ? own > 56 : own < 48) return false;
    }
    if (K == 1 && N <= 2 && own < 58 && t.total >= 16384) return false;
    if (half && K > 2 && K <= 5 && N < 2 * K && t.total > 4800 && t.total <= 6144) return false;
    const double least = 8e6 * (K == 1 || K > 8 ? 8 : K) * (many ? 0.5 : own < 50 ? 2.0 : 1.0);
    return t.total >= kSectorMinTiles && 4.0 * static_cast<double>(G) * D * (K + N) >= least;
}

template <int K>
int run_encode_k(const float *d_queries, float *d_coded, int64_t G, int N, int64_t D, const Nodes &nodes,
                 hipStream_t stream) {
    if (sector_rows(d_queries, d_coded, G, K, N, D)) {
        if constexpr (K >= kMfmaWideMinK) {
            // as for whole rows (run_encode_wide), but where rows of one or two tiles leave the matrix cores' workgroups less to
            // do, only in few tiles (K = 12, N = 28, 300 MB, 156 floats 85 us and 73 without matrix cores,
            // 258 floats 107 and 90, 350 floats 73 and 77).  A call of few tiles is one workgroup's chain, which four waves share: K = 11, N = 26,
            // one row of 218 floats 7.7 and 13.5 us, K = 8, N = 9, 100 rows of 129 floats 0.6 of the time.
            const bool few = sector_tiles(G, D, kTileHalo).total <= (N >= 2 * K + 4 ? 2 * kSectorFewTiles : kSectorFewTiles);
            if (K >= kMfmaMinK || few || (N >= 2 * K + 4 && D >= kMfmaSectorsMinD))
                return run_encode_mfma_sectors<(K + 3) / 4>(d_queries, d_coded, G, K, N, D, nodes, stream);
        }
        if constexpr (K < kMfmaMinK) return run_encode_sectors<K>(d_queries, d_coded, G, N, D, nodes, stream);
    }
    const bool aligned16 = (reinterpret_cast<uintptr_t>(d_queries) % 16 == 0) &&
                           (reinterpret_cast<uintptr_t>(d_coded) % 16 == 0) && (D % 4 == 0);
    if (aligned16) return run_encode_wide<K>(d_queries, d_coded, G, N, D, nodes, stream);
    // rows only 4-byte aligned: 128-bit accesses on the first 4 * (D / 4) columns, 4-byte accesses on the rest;
    // short ragged rows: aligned 64-bit accesses throughout where the rows allow them, else 4-byte accesses
    const int64_t tail = D % 4;
    if constexpr (K >= kMfmaWideMinK) {
        // The matrix-core kernel takes a row's partial last vector along, in rows of any length.  Over 260 calls (where the rows had
        // 4-byte accesses, or a launch of their own for the last columns): K > 16 1.0 to 2.6 times as fast (K = 40, N = 46, 7 x 151 floats
        // 28.7 and 11.2 us; K = 23, N = 57, 15397 x 5 32.9 and 18.6; K = 37, N = 41, 16384 x 151 266 and 248), but for short rows of K < 20
        // queries and hardly more workers in many groups (K = 17, N = 18, 1749 x 49 7.4 and 8.2); K = 9..16 with N >= 2 K + 4 0.97 to 1.7 (K =
        // 16, N = 44, 11677 x 9 27.3 and 16.0; not many rows of 5 to 7, K = 14, N = 37, 9611 x 6 12.9 and 13.9), K = 8 in short rows 0.93
        // to 1.07.
        const bool scalar = tail != 0 && D <= kScalarRowsMaxD && (K == 8 || (K < 20 && 4 * N < 5 * K && G * D > 65536) ||
                                                                   (K < kMfmaMinK && D < 8 && G > 4096));
        if (D >= 4 && !scalar && (K >= kMfmaMinK || N >= 2 * K + 4))
            return run_encode_mfma<(K + 3) / 4, true>(d_queries, d_coded, G, K, N, D, nodes, stream);
    }
    if (tail != 0 && D <= kScalarRowsMaxD) {
        if (D % 2 == 0 && reinterpret_cast<uintptr_t>(d_queries) % 8 == 0 && reinterpret_cast<uintptr_t>(d_coded) % 8 == 0)
            return run_encode<K, 2, false>(d_queries, d_coded, G, N, D, D / 2, 0, nodes, stream);
        return run_encode<K, 1, false>(d_queries, d_coded, G, N, D, D, 0, nodes, stream);
    }
    if constexpr (K < kMfmaMinK) {
        if (D >= 4) {
            const int rc = run_encode<K, 4, true>(d_queries, d_coded, G, N, D, D / 4, 0, nodes, stream);
            if (rc != APPROXIFER_OK || tail == 0) return rc;
        }
        return run_encode<K, 1, false>(d_queries, d_coded, G, N, D, tail, D - tail, nodes, stream);
    }
    return APPROXIFER_ERR_LIMIT;                              // not reached: from kMfmaMinK on every row has gone one of the ways above
}

}  // namespace

// Rows Q .. Q + fill - 1 of a [rows][D] query buffer become copies of row Q - 1 (a stream whose length is not a
// multiple of K: the last group is completed by repeating its last query).  One float per thread.
__global__ void pad_last_group_kernel(float *__restrict__ queries, int64_t Q, int64_t D, int64_t fill) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= fill * D) return;
    const int64_t d = i % D;
    queries[Q * D + i] = queries[(Q - 1) * D + d];
}

int launch_pad_last_group(float *d_queries, int64_t Q, int K, int64_t D, hipStream_t stream) {
    const int64_t fill = (K - Q % K) % K;
    if (fill == 0 || D == 0) return APPROXIFER_OK;
    const int threads = 256;
    const int64_t blocks = (fill * D + threads - 1) / threads;
    if (blocks > 0x7fffffffLL) return APPROXIFER_ERR_LIMIT;
    return launch_status(launch_kernel(pad_last_group_kernel, dim3(static_cast<unsigned>(blocks)), dim3(threads), 0, stream,
                                       d_queries, Q, D, fill));
}

#define APPROXIFER_K_CASE(k) \
    case k: return run_encode_k<k>(d_queries, d_coded, G, N, D, nodes, stream);
#define APPROXIFER_K_CASE8(b)                                                                        \
    APPROXIFER_K_CASE(b + 1) APPROXIFER_K_CASE(b + 2) APPROXIFER_K_CASE(b + 3) APPROXIFER_K_CASE(b + 4) \
    APPROXIFER_K_CASE(b + 5) APPROXIFER_K_CASE(b + 6) APPROXIFER_K_CASE(b + 7) APPROXIFER_K_CASE(b + 8)

int launch_encode(const float *d_queries, float *d_coded, int64_t G, int K, int N, int64_t D, const Nodes &nodes,
                  hipStream_t stream) {
    static_assert(APPROXIFER_MAX_K == 64, "the K dispatch below covers 1..64");
    switch (K) {
        APPROXIFER_K_CASE8(0)
        APPROXIFER_K_CASE8(8)
        APPROXIFER_K_CASE8(16)
        APPROXIFER_K_CASE8(24)
        APPROXIFER_K_CASE8(32)
        APPROXIFER_K_CASE8(40)
        APPROXIFER_K_CASE8(48)
        APPROXIFER_K_CASE8(56)
        default: return APPROXIFER_ERR_LIMIT;
    }
}

}  // namespace approxifer

// What the Byzantine decoder's kernels share: the tail of a group (vote -> located adversaries -> survivors -> decode),
// the meeting of workgroups that share a group, and full-precision reciprocals and roots of normal doubles.
#pragma once

#include "decode_common.h"

namespace approxifer {

// ------------------------------------------------------------------------------------------------
// shared tail: vote -> located adversaries -> F -> decode
// ------------------------------------------------------------------------------------------------
// Decoder contraction of one group over every column tile, predictions read from global memory.
template <int VEC>
__device__ __forceinline__ void contract_group(const float *__restrict__ pg, float *__restrict__ og, const int *F, int nF,
                                               int K, int KP, int64_t C, int64_t Cv, const double *WdT) {
    for (int64_t cv0 = 0; cv0 < Cv; cv0 += kColsPerTile) {
        const int64_t cv1 = (cv0 + kColsPerTile < Cv) ? cv0 + kColsPerTile : Cv;
        typename PredVec<VEC>::type unused[kRowChunk];
        contract_tile<VEC, false>(pg, og, F, nF, K, KP, C, cv0, cv1, WdT, unused);
    }
}

// The A most voted workers (equal counts: smaller index first) go to adv_g in ascending order; F = the
// available workers without them (ascending), Fpos = their positions in `avail`.  n <= 64, N <= 128.
// One wave does it in registers: lane i ranks workers i and i + 64 by counting against the vote counts
// (broadcast reads of LDS), ballots turn ranks into the ascending lists.
// select_adversaries_wave: called by one whole wave after every vote has been added and a barrier; the lists are
// visible after the next barrier.
__device__ __forceinline__ void select_adversaries_wave(int32_t *__restrict__ adv_g, const int *avail, int n, int N,
                                                        int A, const int *votes, int *F, int *Fpos) {
    {
        const int lane = lane_id();
        const int mine0 = lane < N ? votes[lane] : -1;
        const int mine1 = lane + kWave < N ? votes[lane + kWave] : -1;
        int rank0 = 0, rank1 = 0;
#pragma unroll 8
        for (int o = 0; o < N; ++o) {
            const int v = votes[o];
            rank0 += (v > mine0 || (v == mine0 && o < lane)) ? 1 : 0;
            rank1 += (v > mine1 || (v == mine1 && o < lane + kWave)) ? 1 : 0;
        }
        const bool s0 = lane < N && rank0 < A;
        const bool s1 = lane + kWave < N && rank1 < A;
        const unsigned long long m0 = __ballot(s0), m1 = __ballot(s1);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (s0) adv_g[__popcll(m0 & below)] = lane;
        if (s1) adv_g[__popcll(m0) + __popcll(m1 & below)] = lane + kWave;
        const int w = lane < n ? avail[lane] : 0;
        const bool dropped = ((w < kWave ? m0 >> w : m1 >> (w - kWave)) & 1ull) != 0ull;
        const bool keep = lane < n && !dropped;
        const unsigned long long mk = __ballot(keep);
        if (keep) {
            const int pos = __popcll(mk & below);
            F[pos] = w;
            Fpos[pos] = lane;
        }
    }
}

// Called by the whole workgroup after every vote has been added and a barrier; ends with a barrier.
__device__ __forceinline__ void select_adversaries(int32_t *__restrict__ adv_g, const int *avail, int n, int N, int A,
                                                   const int *votes, int *F, int *Fpos) {
    if (wave_id() == 0) select_adversaries_wave(adv_g, avail, n, N, A, votes, F, Fpos);
    __syncthreads();
}

// Several workgroups share a group (few groups, many classes: each takes part of the classes).  They meet in the
// group's N+1 words of the caller's workspace -- N vote counters and an arrival counter, cleared by
// clear_workspace_kernel before the launch.  These words are touched by device-scope atomic read-modify-writes only,
// which are carried out at the one place all workgroups of the device share.  A part's additions have been carried
// out once their old values are back; only then does it count itself in, and the part that counts itself in last
// reads the votes with the same kind of operation: no cache write-back or invalidation (a fence) is needed, and none
// of the part's other memory traffic has to be ordered with this.  No part waits for another: whichever arrives last
// gets every vote (into `votes`, LDS) and true, and finishes the group.
// Called by the whole workgroup after a barrier that follows its last vote; ends with a barrier when it returns true.
__device__ __forceinline__ bool pool_votes_last_arrival(int *gvotes, int *votes, int N, int splits, int *flag) {
    const int tid = threadIdx.x;
    int seen = 0;
    for (int i = tid; i < N; i += blockDim.x)
        if (votes[i] != 0) seen |= __hip_atomic_fetch_add(&gvotes[i], votes[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(seen));                         // the returned values are waited for
    __syncthreads();
    if (tid == 0)
        *flag = __hip_atomic_fetch_add(&gvotes[N], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == splits - 1 ? 1 : 0;
    __syncthreads();
    if (*flag == 0) return false;
    for (int i = tid; i < N; i += blockDim.x)
        votes[i] = __hip_atomic_fetch_add(&gvotes[i], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return true;
}

// vec4: prediction rows are 16-byte aligned and C % 4 == 0, Cv = C / 4; else Cv = C.
__device__ __forceinline__ void finish_group(const float *__restrict__ pg, float *__restrict__ og,
                                             int32_t *__restrict__ adv_g, const int *avail, int n, int N, int A, int K,
                                             int KP, int64_t C, int64_t Cv, bool vec4, int sign_mode,
                                             const double *alpha_s, const double *beta_s, const int *votes,
                                             int *F, int *Fpos, double *WdT) {
    select_adversaries(adv_g, avail, n, N, A, votes, F, Fpos);
    const int nF = n - A;
    decoder_weights(alpha_s, beta_s, F, nF, K, KP, sign_mode, WdT);
    __syncthreads();
    if (vec4) contract_group<4>(pg, og, F, nF, K, KP, C, Cv, WdT);
    else contract_group<1>(pg, og, F, nF, K, KP, C, Cv, WdT);
}

// Reciprocal and square root of a normal, positive-or-negative (rcp) / positive (sqrt) double to full
// double precision: the hardware estimate refined by two Newton (Goldschmidt) steps and, for the root, one
// residual correction.  No scaling for denormals or infinities and no final correctly-rounded fix-up, which
// the factorisations here do not need: their operands are column norms and pivots, and a zero norm is
// handled by the caller.
__device__ __forceinline__ double rcp_normal(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}
__device__ __forceinline__ double sqrt_normal(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, s), h, g);
}

__device__ __forceinline__ double rsqrt_normal(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    return 2.0 * fma(h, r, h);
}

}  // namespace approxifer

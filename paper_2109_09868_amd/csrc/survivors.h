// The list of a group's survivors that the 16-lane row kernels go over, N <= 64 workers: one byte per entry.  Plain
// functions of the mask bits and the lane, so that a host program can check which workers a list names.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace approxifer {

constexpr int kListLanes = 16;
// 64 workers and the overhang of the last pass: passes take up to sixteen entries, from multiples of 8, 12 or 16 below 64.
constexpr int kListBytes = 80;

// First every entry names the first survivor, four entries to a store ..
__host__ __device__ inline void list_first(unsigned long long m, uint8_t *F, int lane) {
    const uint32_t first = m != 0ull ? static_cast<uint32_t>(__builtin_ctzll(m)) : 0u;
    uint32_t *w = reinterpret_cast<uint32_t *>(F);
    for (int e = lane; e < kListBytes / 4; e += kListLanes) w[e] = first * 0x01010101u;
}
// .. then survivor i takes entry number (survivors below i).
__host__ __device__ inline void list_ranks(unsigned long long m, uint8_t *F, int lane) {
    for (int p = 0; p < 4; ++p) {
        const int i = p * kListLanes + lane;
        if ((m >> i) & 1ull) F[__builtin_popcountll(m & ((1ull << i) - 1ull))] = static_cast<uint8_t>(i);
    }
}

}  // namespace approxifer

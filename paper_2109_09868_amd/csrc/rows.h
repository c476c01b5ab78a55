// Operations along a row of 16 lanes: broadcasts of one lane's double, and multiply-adds that take their first factor
// from another lane of the row.
#pragma once

#include "common.h"

namespace approxifer {

template <int LANE>
__device__ __forceinline__ double row_bcast(double v) {   // lane LANE of every 16-lane row, to the whole row
    // all rows and banks enabled and every source lane exists: the 'old' operand is never used, and with
    // bound_ctrl set the compiler knows it and does not materialise it
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + LANE, 0xF, 0xF, true);
}

// The same for a lane index that is only known after unrolling.
__device__ __forceinline__ double row_bcast_dyn(double v, int lane_in_row) {
    switch (lane_in_row) {
        case 0: return row_bcast<0>(v);
        case 1: return row_bcast<1>(v);
        case 2: return row_bcast<2>(v);
        case 3: return row_bcast<3>(v);
        case 4: return row_bcast<4>(v);
        case 5: return row_bcast<5>(v);
        case 6: return row_bcast<6>(v);
        case 7: return row_bcast<7>(v);
        case 8: return row_bcast<8>(v);
        case 9: return row_bcast<9>(v);
        case 10: return row_bcast<10>(v);
        case 11: return row_bcast<11>(v);
        case 12: return row_bcast<12>(v);
        case 13: return row_bcast<13>(v);
        case 14: return row_bcast<14>(v);
        default: return row_bcast<15>(v);
    }
}

// v_fmac_f64 takes its first factor from one lane of the row by itself (row_newbcast), at the rate of a plain
// v_fmac_f64 (4 cycles per wave measured for either); the compiler spends a 64-bit move per broadcast instead.  Passes
// over a column are therefore written out.  A DPP operand must not be read within two wait states of the VALU
// instruction that wrote it, and the compiler does not see into a block: each opens with s_nop 1, and inside no
// instruction reads what an earlier one wrote as its DPP operand.  Nor may a block read what a matrix instruction wrote
// (up to 19 wait states that only the compiler inserts): nothing here does.

// a[O + i] += bcast_i(u) * p: an outer product, lane i of the row holding the first factor of element i
#define APX_O(x, i) "v_fmac_f64_dpp %[" #x "], %[u], %[p] row_newbcast:%[" #i "] row_mask:0xf bank_mask:0xf\n"
template <int O, int L, int CNT, int RM>
__device__ __forceinline__ void row_outer(double (&a)[RM], double u, double p) {
    if constexpr (CNT >= 8) {
        asm("s_nop 1\n" APX_O(a0, i0) APX_O(a1, i1) APX_O(a2, i2) APX_O(a3, i3) APX_O(a4, i4) APX_O(a5, i5) APX_O(a6, i6)
                APX_O(a7, i7)
            : [a0] "+v"(a[O]), [a1] "+v"(a[O + 1]), [a2] "+v"(a[O + 2]), [a3] "+v"(a[O + 3]), [a4] "+v"(a[O + 4]),
              [a5] "+v"(a[O + 5]), [a6] "+v"(a[O + 6]), [a7] "+v"(a[O + 7])
            : [u] "v"(u), [p] "v"(p), [i0] "n"(L), [i1] "n"(L + 1), [i2] "n"(L + 2), [i3] "n"(L + 3), [i4] "n"(L + 4),
              [i5] "n"(L + 5), [i6] "n"(L + 6), [i7] "n"(L + 7));
        row_outer<O + 8, L + 8, CNT - 8>(a, u, p);
    } else if constexpr (CNT >= 2) {
        asm("s_nop 1\n" APX_O(a0, i0) APX_O(a1, i1)
            : [a0] "+v"(a[O]), [a1] "+v"(a[O + 1])
            : [u] "v"(u), [p] "v"(p), [i0] "n"(L), [i1] "n"(L + 1));
        row_outer<O + 2, L + 2, CNT - 2>(a, u, p);
    } else if constexpr (CNT == 1) {
        asm("s_nop 1\n" APX_O(a0, i0) : [a0] "+v"(a[O]) : [u] "v"(u), [p] "v"(p), [i0] "n"(L));
    }
}
#undef APX_O

}  // namespace approxifer

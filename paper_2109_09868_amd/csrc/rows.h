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
// (up to 19 wait states that only the compiler inserts): nothing here does.  What a block writes is marked early-clobber:
// it is written before the block has read its last factor, and an accumulator that starts out equal to a factor (a zero,
// say) would otherwise be given the factor's register.

// a[O + i] += bcast_i(u) * p: an outer product, lane i of the row holding the first factor of element i
#define APX_O(x, i) "v_fmac_f64_dpp %[" #x "], %[u], %[p] row_newbcast:%[" #i "] row_mask:0xf bank_mask:0xf\n"
template <int O, int L, int CNT, int RM>
__device__ __forceinline__ void row_outer(double (&a)[RM], double u, double p) {
    if constexpr (CNT >= 8) {
        asm("s_nop 1\n" APX_O(a0, i0) APX_O(a1, i1) APX_O(a2, i2) APX_O(a3, i3) APX_O(a4, i4) APX_O(a5, i5) APX_O(a6, i6)
                APX_O(a7, i7)
            : [a0] "+&v"(a[O]), [a1] "+&v"(a[O + 1]), [a2] "+&v"(a[O + 2]), [a3] "+&v"(a[O + 3]), [a4] "+&v"(a[O + 4]),
              [a5] "+&v"(a[O + 5]), [a6] "+&v"(a[O + 6]), [a7] "+&v"(a[O + 7])
            : [u] "v"(u), [p] "v"(p), [i0] "n"(L), [i1] "n"(L + 1), [i2] "n"(L + 2), [i3] "n"(L + 3), [i4] "n"(L + 4),
              [i5] "n"(L + 5), [i6] "n"(L + 6), [i7] "n"(L + 7));
        row_outer<O + 8, L + 8, CNT - 8>(a, u, p);
    } else if constexpr (CNT >= 2) {
        asm("s_nop 1\n" APX_O(a0, i0) APX_O(a1, i1)
            : [a0] "+&v"(a[O]), [a1] "+&v"(a[O + 1])
            : [u] "v"(u), [p] "v"(p), [i0] "n"(L), [i1] "n"(L + 1));
        row_outer<O + 2, L + 2, CNT - 2>(a, u, p);
    } else if constexpr (CNT == 1) {
        asm("s_nop 1\n" APX_O(a0, i0) : [a0] "+&v"(a[O]) : [u] "v"(u), [p] "v"(p), [i0] "n"(L));
    }
}
#undef APX_O

// Passes over a column, lane LANE of the row holding the first factors:
//     row_dot:   d0, d1 += bcast(a[r]) * b[r]     (even and odd r: two chains)
//     row_axpy:  a[r]   += bcast(b[r]) * f
// `b` may be `a` itself: every element is read before it is written, once.
#define APX_DPP " row_newbcast:%[l] row_mask:0xf bank_mask:0xf\n"
#define APX_D2(x, y, u, v) "v_fmac_f64_dpp %[d0], %[" #x "], %[" #u "]" APX_DPP "v_fmac_f64_dpp %[d1], %[" #y "], %[" #v "]" APX_DPP
#define APX_U(x, u) "v_fmac_f64_dpp %[" #x "], %[" #u "], %[f]" APX_DPP
template <int LANE, int O, int RM>
__device__ __forceinline__ void row_dot2(const double (&a)[RM], const double (&b)[RM], double &d0, double &d1) {
    asm("s_nop 1\n" APX_D2(a0, a1, b0, b1)
        : [d0] "+&v"(d0), [d1] "+&v"(d1)
        : [a0] "v"(a[O]), [a1] "v"(a[O + 1]), [b0] "v"(b[O]), [b1] "v"(b[O + 1]), [l] "n"(LANE));
}
template <int LANE, int O, int RM>
__device__ __forceinline__ void row_dot4(const double (&a)[RM], const double (&b)[RM], double &d0, double &d1) {
    asm("s_nop 1\n" APX_D2(a0, a1, b0, b1) APX_D2(a2, a3, b2, b3)
        : [d0] "+&v"(d0), [d1] "+&v"(d1)
        : [a0] "v"(a[O]), [a1] "v"(a[O + 1]), [a2] "v"(a[O + 2]), [a3] "v"(a[O + 3]), [b0] "v"(b[O]), [b1] "v"(b[O + 1]),
          [b2] "v"(b[O + 2]), [b3] "v"(b[O + 3]), [l] "n"(LANE));
}
template <int LANE, int O, int RM>
__device__ __forceinline__ void row_dot8(const double (&a)[RM], const double (&b)[RM], double &d0, double &d1) {
    asm("s_nop 1\n" APX_D2(a0, a1, b0, b1) APX_D2(a2, a3, b2, b3) APX_D2(a4, a5, b4, b5) APX_D2(a6, a7, b6, b7)
        : [d0] "+&v"(d0), [d1] "+&v"(d1)
        : [a0] "v"(a[O]), [a1] "v"(a[O + 1]), [a2] "v"(a[O + 2]), [a3] "v"(a[O + 3]), [a4] "v"(a[O + 4]),
          [a5] "v"(a[O + 5]), [a6] "v"(a[O + 6]), [a7] "v"(a[O + 7]), [b0] "v"(b[O]), [b1] "v"(b[O + 1]),
          [b2] "v"(b[O + 2]), [b3] "v"(b[O + 3]), [b4] "v"(b[O + 4]), [b5] "v"(b[O + 5]), [b6] "v"(b[O + 6]),
          [b7] "v"(b[O + 7]), [l] "n"(LANE));
}
template <int LANE, int O, int RM>
__device__ __forceinline__ void row_dot(const double (&a)[RM], const double (&b)[RM], double &d0, double &d1) {
    if constexpr ((RM - O) % 2 == 1) {                    // an odd row first, then whole pairs
        asm("s_nop 1\n v_fmac_f64_dpp %[d0], %[a0], %[b0]" APX_DPP
            : [d0] "+&v"(d0)
            : [a0] "v"(a[O]), [b0] "v"(b[O]), [l] "n"(LANE));
        row_dot<LANE, O + 1>(a, b, d1, d0);
    } else if constexpr (RM - O >= 8) {
        row_dot8<LANE, O>(a, b, d0, d1);
        row_dot<LANE, O + 8>(a, b, d0, d1);
    } else if constexpr (RM - O >= 4) {
        row_dot4<LANE, O>(a, b, d0, d1);
        row_dot<LANE, O + 4>(a, b, d0, d1);
    } else if constexpr (RM - O >= 2) {
        row_dot2<LANE, O>(a, b, d0, d1);
    }
}
// a[r] += bcast(a[r]) * f
template <int LANE, int O, int RM>
__device__ __forceinline__ void row_axpy_self(double (&a)[RM], double f) {
    if constexpr (RM - O >= 8) {
        asm("s_nop 1\n" APX_U(a0, a0) APX_U(a1, a1) APX_U(a2, a2) APX_U(a3, a3) APX_U(a4, a4) APX_U(a5, a5)
                APX_U(a6, a6) APX_U(a7, a7)
            : [a0] "+&v"(a[O]), [a1] "+&v"(a[O + 1]), [a2] "+&v"(a[O + 2]), [a3] "+&v"(a[O + 3]), [a4] "+&v"(a[O + 4]),
              [a5] "+&v"(a[O + 5]), [a6] "+&v"(a[O + 6]), [a7] "+&v"(a[O + 7])
            : [f] "v"(f), [l] "n"(LANE));
        row_axpy_self<LANE, O + 8>(a, f);
    } else if constexpr (RM - O >= 4) {
        asm("s_nop 1\n" APX_U(a0, a0) APX_U(a1, a1) APX_U(a2, a2) APX_U(a3, a3)
            : [a0] "+&v"(a[O]), [a1] "+&v"(a[O + 1]), [a2] "+&v"(a[O + 2]), [a3] "+&v"(a[O + 3])
            : [f] "v"(f), [l] "n"(LANE));
        row_axpy_self<LANE, O + 4>(a, f);
    } else if constexpr (RM - O >= 2) {
        asm("s_nop 1\n" APX_U(a0, a0) APX_U(a1, a1)
            : [a0] "+&v"(a[O]), [a1] "+&v"(a[O + 1])
            : [f] "v"(f), [l] "n"(LANE));
        row_axpy_self<LANE, O + 2>(a, f);
    } else if constexpr (RM - O == 1) {
        asm("s_nop 1\n" APX_U(a0, a0) : [a0] "+&v"(a[O]) : [f] "v"(f), [l] "n"(LANE));
    }
}
// q[r] += bcast(b[r]) * f for r < T
template <int LANE, int O, int T, int NQ, int NB>
__device__ __forceinline__ void row_axpy(double (&q)[NQ], const double (&b)[NB], double f) {
    if constexpr (T - O >= 4) {
        asm("s_nop 1\n" APX_U(q0, b0) APX_U(q1, b1) APX_U(q2, b2) APX_U(q3, b3)
            : [q0] "+&v"(q[O]), [q1] "+&v"(q[O + 1]), [q2] "+&v"(q[O + 2]), [q3] "+&v"(q[O + 3])
            : [b0] "v"(b[O]), [b1] "v"(b[O + 1]), [b2] "v"(b[O + 2]), [b3] "v"(b[O + 3]), [f] "v"(f), [l] "n"(LANE));
        row_axpy<LANE, O + 4, T>(q, b, f);
    } else if constexpr (T - O >= 1) {
        asm("s_nop 1\n" APX_U(q0, b0) : [q0] "+&v"(q[O]) : [b0] "v"(b[O]), [f] "v"(f), [l] "n"(LANE));
        row_axpy<LANE, O + 1, T>(q, b, f);
    }
}
// One step of a triangular sweep: s and t gain their multiples of entry LANE of s, which is final (f is 0 there).
template <int LANE>
__device__ __forceinline__ void row_sweep(double &s, double f) {
    asm("s_nop 1\n v_fmac_f64_dpp %[s], %[s], %[f]" APX_DPP : [s] "+&v"(s) : [f] "v"(f), [l] "n"(LANE));
}
template <int LANE>
__device__ __forceinline__ void row_sweep2(double &s, double f, double &t, double b) {
    asm("s_nop 1\n v_fmac_f64_dpp %[t], %[s], %[b]" APX_DPP "v_fmac_f64_dpp %[s], %[s], %[f]" APX_DPP
        : [s] "+&v"(s), [t] "+&v"(t)
        : [f] "v"(f), [b] "v"(b), [l] "n"(LANE));
}
#undef APX_U
#undef APX_D2
#undef APX_DPP

}  // namespace approxifer

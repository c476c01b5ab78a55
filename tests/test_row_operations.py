"""The hand-written multiply-add blocks of csrc/rows.h: an instruction of a block must not read, as a factor, a register that
an earlier one of the same block has written.  The compiler may give an accumulator and a factor one register where it can
prove that they start out equal, unless the block says that it writes the accumulator before it has read its factors
(early clobber).  The probes below make them equal; the assembly of these probes is looked at."""
import re
import subprocess

PROBE = r"""
#include "rows.h"
using namespace approxifer;
extern "C" __global__ void outer(const double *in, double *out) {          // accumulators that start as the factors
    const double u = in[threadIdx.x], p = in[threadIdx.x + 64];
    double a[11], b[11];
#pragma unroll
    for (int i = 0; i < 11; ++i) { a[i] = p; b[i] = u; }
    row_outer<0, 0, 11>(a, u, p);
    row_outer<0, 0, 11>(b, u, p);
#pragma unroll
    for (int i = 0; i < 11; ++i) out[threadIdx.x + 64 * i] = a[i] + 2.0 * b[i];
}
extern "C" __global__ void dot(const double *in, double *out) {            // sums that start as elements of the columns
    double a[15], b[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) { a[i] = in[threadIdx.x + 64 * i]; b[i] = in[threadIdx.x + 64 * (15 + i)]; }
    double d0 = a[3], d1 = b[5], e0 = b[14], e1 = a[14];
    row_dot<2, 0>(a, b, d0, d1);
    row_dot<3, 1>(a, b, e0, e1);
    out[threadIdx.x] = d0 + 2.0 * d1 + 3.0 * e0 + 4.0 * e1;
    double z0 = 0.0, z1 = 0.0;
    double c[8] = {0.0, a[0], 0.0, a[1], a[2], 0.0, 0.0, a[3]};
    row_dot<1, 0>(c, c, z0, z1);
    out[threadIdx.x + 64] = z0 - z1;
}
extern "C" __global__ void axpy(const double *in, double *out) {           // columns that hold the factor or each other
    const double f = in[threadIdx.x];
    double a[15], q[15], b[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) { a[i] = f; b[i] = in[threadIdx.x + 64 * i]; q[i] = i < 14 ? b[i + 1] : f; }
    row_axpy_self<2, 0>(a, f);
    row_axpy<3, 0, 15>(q, b, f);
#pragma unroll
    for (int i = 0; i < 15; ++i) out[threadIdx.x + 64 * i] = a[i] + 2.0 * q[i];
}
extern "C" __global__ void sweep(const double *in, double *out) {
    const double x = in[threadIdx.x], y = in[threadIdx.x + 64];
    double s = x, t = y, v = x, w = x;
    row_sweep2<2>(s, y, t, x);
    row_sweep2<3>(v, x, w, y);
    out[threadIdx.x] = s + 2.0 * t + 3.0 * v + 4.0 * w;
}
"""


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1))


def test_no_block_reads_a_factor_that_it_has_already_overwritten(tmp_path):
    from paper_2109_09868_amd import build
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run([build.hipcc_path(), *build.HIPCC_FLAGS, "-I", build.ROOT + "/include", "-I", build.CSRC, "-S", "--cuda-device-only",
                    str(src), "-o", str(asm)], check=True, capture_output=True)
    blocks = re.findall(r";#ASMSTART\n(.*?);#ASMEND", asm.read_text(), re.S)
    seen = 0
    for block in blocks:
        written = set()
        for line in block.splitlines():
            m = re.match(r"\s*v_fmac_f64_dpp (\S+), (\S+), (\S+) row_newbcast", line)
            if not m:
                assert line.strip() in ("", ";", "s_nop 1"), line
                continue
            dst, f0, f1 = (_registers(g) for g in m.groups())
            assert not written & (f0 | f1), block
            written |= dst
            seen += 1
    assert seen > 80

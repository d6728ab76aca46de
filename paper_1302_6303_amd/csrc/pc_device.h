// Arithmetic shared by the preconditioner's kernels.  The same cell may be
// relaxed by kernels over native, colour-split or LDS storage, and their
// results agree bit for bit: every operation is written out here, without
// contraction (fused multiply-adds only where they are written).
#pragma once

#include "device_util.h"

namespace nrd {

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) {
    return __builtin_fma(a, b, c);
}

// Diagonal term of E on a Marshak face with boundary coefficient Db.
template <typename PT>
__device__ __forceinline__ PT robin_diag(PT beta, PT Db, PT h) {
#pragma clang fp contract(off)
    return PT(2) * beta * Db / (fma_t(PT(4), Db, h) * h);
}

// One cell of a Gauss-Seidel half-sweep.
template <typename PT>
__device__ __forceinline__ PT relax(PT f, PT ns, PT dg) {
#pragma clang fp contract(off)
    return div_pos(f + ns, dg);
}

// Residual of one cell's equation.
template <typename PT>
__device__ __forceinline__ PT cell_residual(PT f, PT ns, PT dg, PT e) {
#pragma clang fp contract(off)
    return f - fma_t(dg, e, -ns);
}

// Trilinear interpolation (weights 3/4, 1/4 per axis) from the coarse values
// s[a][b][c], 0: the cell's own coarse index on that axis, 1: its neighbour's.
template <typename PT>
__device__ __forceinline__ PT trilinear(const PT s[2][2][2]) {
#pragma clang fp contract(off)
    PT v = PT(0);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const PT w = (a ? PT(0.25) : PT(0.75)) * (b ? PT(0.25) : PT(0.75)) *
                             (c ? PT(0.25) : PT(0.75));
                v = fma_t(w, s[a][b][c], v);
            }
    return v;
}

// P2^-1 of one cell: [[1 + sigma beta, -k beta z^3], [-sigma beta, 1 + k beta
// z^3]] (sigma T^3 = z^3), or of its transpose.
__device__ __forceinline__ void p2_cell(double sg, double z, double beta, int mode, int transpose,
                                        double eE, double eT, double& yE, double& yT) {
#pragma clang fp contract(off)
    const double k = mode ? 4.0 : 1.0;
    const double a = fma_t(sg, beta, 1.0), b = -k * beta * z, cc = -sg * beta,
                 d = fma_t(k * beta, z, 1.0);
    const double det = fma_t(a, d, -(b * cc));
    if (!transpose) {
        yE = div_pos(fma_t(d, eE, -(b * eT)), det);
        yT = div_pos(fma_t(a, eT, -(cc * eE)), det);
    } else {
        yE = div_pos(fma_t(d, eE, -(cc * eT)), det);
        yT = div_pos(fma_t(a, eT, -(b * eE)), det);
    }
}

}  // namespace nrd

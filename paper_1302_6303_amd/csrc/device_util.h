// Device helpers shared by the stencil and transpose kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace nrd {

// Reciprocal and reciprocal square root: the hardware estimate (about 24
// correct bits) refined by one step of third order or two of Newton-Raphson
// (the result is within about one ulp); valid for the positive, normal operands
// met here.  The reciprocal, and the root below, give the same bits either way
// over 2^22 operands; one step takes one and three operations less
// (preconditioner of 96^3 185.9 -> 183.4 us).
__device__ __forceinline__ double rcp_nr(double x) {
    // one step of third order: y (1 + e + e^2), e = 1 - x y of 24 bits
    const double y = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, __builtin_fma(e, e, e), y);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double r = __builtin_fma(-(x * y), y, 1.0);     // y <- y (3 - x y^2) / 2
    y = __builtin_fma(0.5 * y, r, y);
    r = __builtin_fma(-(x * y), y, 1.0);
    return __builtin_fma(0.5 * y, r, y);
}

// Interior cell (i, j, k) of the linear (x fastest) interior index lin of
// patch p, and the native (ghosted) index of an interior cell.
__device__ __forceinline__ void cell_coords(const PatchInfo& p, int lin, int& i, int& j,
                                            int& k) {
    i = lin % p.n[0];
    const int r = lin / p.n[0];
    j = r % p.n[1];
    k = r / p.n[1];
}

__device__ __forceinline__ int native_index(const PatchInfo& p, int i, int j, int k) {
    return p.off + (i + 1) + p.sy * (j + 1) + p.sz * (k + 1);
}

// Quotient by d > 0, infinite and NaN operands included, and square root of a
// finite x >= 0: the hardware estimate refined until the last correction is
// below an ulp; the library's forms take up to three times the instructions.
// Over 2^22 operands of each type no quotient differed from the correctly
// rounded one for divisors from 1 to the largest finite one (subnormal ones: by
// an ulp, rarely), nor a root from 1e-33 (double: 1e-296) on.  A smaller root is
// off, but face_DT, its caller, multiplies it by kappa x^2: no product differed
// over 2^22 pairs of x and kappa, subnormal ones included.  The sweeps of the
// base grid are bound by instruction issue: 96^3 in double 248 -> 226 us per
// preconditioner, 128^3 in float 14.5 -> 13.8 ms per four steps (divisors beyond
// 2^126 and infinities among them at no cost: 182.4 us and 12.7 ms either way).
__device__ __forceinline__ float sqrt_pos(float x) {
    const float y = __builtin_amdgcn_rsqf(x + 1e-37f);   // finite at 0
    const float g = x * y;
    return __builtin_fmaf(__builtin_fmaf(-g, g, x), 0.5f * y, g);
}
__device__ __forceinline__ double sqrt_pos(double x) {
    // 1 / sqrt(x) by one step of third order, y (1 + r / 2 + 3 r^2 / 8)
    double y = __builtin_amdgcn_rsq(x + 1e-300);
    const double r = __builtin_fma(-(x * y), y, 1.0);
    y = __builtin_fma(y, r * __builtin_fma(0.375, r, 0.5), y);
    const double g = x * y;
    return __builtin_fma(__builtin_fma(-g, g, x), 0.5 * y, g);
}
__device__ __forceinline__ float div_pos(float n, float d) {
    // (the estimate of d / 4: that of d itself is flushed to 0 beyond 2^126)
    const float d4 = 0.25f * d;
    float y = __builtin_amdgcn_rcpf(d4);
    y = 0.25f * __builtin_fmaf(__builtin_fmaf(-d4, y, 1.0f), y, y);
    const float q = n * y;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d, q, n), y, q), d, n);
}
__device__ __forceinline__ double div_pos(double n, double d) {
    const double y = rcp_nr(d);
    const double q = n * y;
    return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-d, q, n), y, q), d, n);
}

// D_T = kappa T_f^(5/2) of the face between cells of temperatures Ta, Tb
// (symmetric in Ta, Tb); the sweeps over colour-split storage recompute it
// from T with this same expression, so they see the snapshot's values.
template <typename PT>
__device__ __forceinline__ PT face_DT(PT Ta, PT Tb, PT kappa) {
#pragma clang fp contract(off)
    const PT Tf = PT(0.5) * (Ta + Tb);
    return kappa * Tf * Tf * sqrt_pos(Tf);
}

}  // namespace nrd

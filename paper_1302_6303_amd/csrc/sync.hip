// Synchronisation of the AMR hierarchy (paper Sec. 3.2.1): covered cells
// take the mean of their eight children (restriction, finest level first);
// ghosts take a sibling patch's value or the coarse-fine interpolation of
// the coarser level (a bilinear tangential stencil of four coarse cells,
// weights 9, 3, 3, 1 over 16, blended 2/3 : 1/3 with the fine cell inside).
// Both are driven by flat host-built tables, one thread per entry.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace nrd {

// One field per blockIdx.y here and below: the tables are small, and what
// bounds these launches is the latency of a thread's own chain of loads (17 k
// ghosts 4.4 -> 2.6 us).  Ghost tables of more blocks than kFieldBlocks are
// bound by their own traffic, which a thread that takes both fields reads once:
// 11 345 blocks 93 -> 89 us, in float 76 -> 72; at 5511 and fewer equal.
constexpr int kFieldBlocks = 8192;

// NF fields per thread, from field NF blockIdx.y on
template <typename T, int NF>
__global__ __launch_bounds__(kBlock) void k_ghost_fill(const GhostCopy* __restrict__ cp,
                                                       int ncp,
                                                       const GhostCF* __restrict__ cf,
                                                       int ncf, T* __restrict__ x,
                                                       int64_t nl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    T* y = x + NF * blockIdx.y * nl;
    if (t < ncp) {
        const GhostCopy e = cp[t];
#pragma unroll
        for (int f = 0; f < NF; ++f) y[f * nl + e.dst] = y[f * nl + e.src];
    } else if (t < ncp + ncf) {
        const GhostCF e = cf[t - ncp];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            T* v = y + f * nl;
            const T ci = (T(9) * v[e.src[0]] + T(3) * v[e.src[1]] + T(3) * v[e.src[2]] +
                          v[e.src[3]]) * T(0.0625);
            v[e.dst] = T(2.0 / 3.0) * ci + T(1.0 / 3.0) * v[e.src[4]];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_restrict(const SyncEntry* __restrict__ se,
                                                     int n, T* __restrict__ x, int64_t nl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const SyncEntry e = se[t];
    T* f = x + blockIdx.y * nl;
    const T* y = f + e.src;
    T acc = y[0];
    acc += y[1];
    acc += y[e.sy];
    acc += y[e.sy + 1];
    acc += y[e.sz];
    acc += y[e.sz + 1];
    acc += y[e.sz + e.sy];
    acc += y[e.sz + e.sy + 1];
    f[e.dst] = acc * T(0.125);
}

static inline int nblocks(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

template <typename T>
static void fill_t(const Dev& D, hipStream_t s, const GhostCopy* cp, int ncp, int ncf, T* x,
                   int nf) {
    const int nb = nblocks((int64_t)ncp + ncf);
    if (nb == 0) return;
    if (nf == 2 && nb > kFieldBlocks)
        k_ghost_fill<T, 2><<<nb, kBlock, 0, s>>>(cp, ncp, D.gcf, ncf, x, D.nl);
    else
        k_ghost_fill<T, 1><<<dim3(nb, nf), kBlock, 0, s>>>(cp, ncp, D.gcf, ncf, x, D.nl);
}

void ghost_fill_d(const Dev& D, hipStream_t s, double* x, int nf) {
    fill_t(D, s, D.gcopy, D.ncopy, D.ncf, x, nf);
}
void ghost_fill_f(const Dev& D, hipStream_t s, float* x, int nf) {
    fill_t(D, s, D.gcopy, D.ncopy, D.ncf, x, nf);
}

template <typename T>
static void restrict_t(const Dev& D, hipStream_t s, T* x, int nf, int lev_lo) {
    for (int l = D.nlev - 2; l >= lev_lo; --l) {
        if (D.nsync[l] == 0) continue;
        k_restrict<T><<<dim3(nblocks(D.nsync[l]), nf), kBlock, 0, s>>>(D.sync[l], D.nsync[l], x,
                                                                       D.nl);
    }
}
void restrict_d(const Dev& D, hipStream_t s, double* x, int nf, int lev_lo) {
    restrict_t<double>(D, s, x, nf, lev_lo);
}
void restrict_f(const Dev& D, hipStream_t s, float* x, int nf, int lev_lo) {
    restrict_t<float>(D, s, x, nf, lev_lo);
}

// Adjoint ghost fill of the two fields of a multiplier vector: sibling
// copies; a coarse-fine ghost takes 1/8 of the coarse cell it lies in.
__global__ __launch_bounds__(kBlock) void k_adjoint_ghost(const GhostCopy* __restrict__ cp,
                                                          int ncp,
                                                          const GhostCF* __restrict__ cf,
                                                          int ncf, double* __restrict__ x,
                                                          int64_t nl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < ncp) {
        const GhostCopy e = cp[t];
        x[e.dst] = x[e.src];
        x[nl + e.dst] = x[nl + e.src];
    } else if (t < ncp + ncf) {
        const GhostCF e = cf[t - ncp];
        x[e.dst] = 0.125 * x[e.src[0]];
        x[nl + e.dst] = 0.125 * x[nl + e.src[0]];
    }
}

// Transposed restriction of one level: a covered cell hands 1/8 of its
// value to each child and keeps none (one field per blockIdx.y; all children
// are loaded before the first is stored: 6.5 -> 4.2 us for 20 k covered cells).
__global__ __launch_bounds__(kBlock) void k_restrict_t(const SyncEntry* __restrict__ se,
                                                       int n, double* __restrict__ x,
                                                       int64_t nl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const SyncEntry e = se[t];
    double* z = x + blockIdx.y * nl;
    double* y = z + e.src;
    const double v = 0.125 * z[e.dst];
    const int64_t at[8] = {0, 1, e.sy, e.sy + 1, e.sz, e.sz + 1, e.sz + e.sy, e.sz + e.sy + 1};
    double c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) c[k] = y[at[k]];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[at[k]] = c[k] + v;
    z[e.dst] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_zero_covered(const SyncEntry* __restrict__ se,
                                                         int n, double* __restrict__ x,
                                                         int nf, int64_t nl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int32_t c = se[t].dst;
    for (int f = 0; f < nf; ++f) x[f * nl + c] = 0.0;
}

void adjoint_ghost_fill(const Dev& D, hipStream_t s, double* x) {
    const int n = D.ncopy + D.ncf;
    if (n == 0) return;
    k_adjoint_ghost<<<nblocks(n), kBlock, 0, s>>>(D.gcopy, D.ncopy, D.gcf, D.ncf, x, D.nl);
}
void restrict_transpose(const Dev& D, hipStream_t s, double* x, int nf) {
    for (int l = 0; l + 1 < D.nlev; ++l) {
        if (D.nsync[l] == 0) continue;
        k_restrict_t<<<dim3(nblocks(D.nsync[l]), nf), kBlock, 0, s>>>(D.sync[l], D.nsync[l], x,
                                                                    D.nl);
    }
}
void zero_covered(const Dev& D, hipStream_t s, double* x, int nf) {
    for (int l = 0; l + 1 < D.nlev; ++l) {
        if (D.nsync[l] == 0) continue;
        k_zero_covered<<<nblocks(D.nsync[l]), kBlock, 0, s>>>(D.sync[l], D.nsync[l], x, nf,
                                                              D.nl);
    }
}

template <typename T>
static void sib_t(const Dev& D, hipStream_t s, T* x, int nf, int lev, int lev_hi) {
    const int a = D.level_sib0[lev], b = D.level_sib0[(lev_hi < 0 ? lev : lev_hi) + 1];
    if (b > a) fill_t(D, s, D.sib + a, b - a, 0, x, nf);
}
void sibling_exchange_f(const Dev& D, hipStream_t s, float* x, int nf, int lev, int lev_hi) {
    sib_t<float>(D, s, x, nf, lev, lev_hi);
}
void sibling_exchange_d(const Dev& D, hipStream_t s, double* x, int nf, int lev, int lev_hi) {
    sib_t<double>(D, s, x, nf, lev, lev_hi);
}

}  // namespace nrd

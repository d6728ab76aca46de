// Krylov vector kernels: per-problem inner products (two-stage, fixed
// order, hence bitwise reproducible), vector combinations, positivity
// reductions and the small per-problem FGMRES kernels (Sec. 4.1).
//
// Vectors are native 2-field arrays; only interior cells are read or
// written.  Inner products are volume weighted over composite cells.
#include <hip/hip_runtime.h>

#include <cfloat>

#include "kernels.h"
#include "precond.h"

namespace nrd {

static inline int nblocks(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

// Sum over the workgroup (4 waves), same result on every thread.
__device__ __forceinline__ double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    const double r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return r;
}
__device__ __forceinline__ double block_min(double v, double* sh) {
    v = wave_min(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    const double r = fmin(fmin(sh[0], sh[1]), fmin(sh[2], sh[3]));
    __syncthreads();
    return r;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double block_max(double v, double* sh) {
    v = wave_max(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    const double r = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    __syncthreads();
    return r;
}

__device__ __forceinline__ int interior_cell(const PatchInfo& p, int lin, int& i, int& j,
                                             int& k) {
    i = lin % p.n[0];
    const int r = lin / p.n[0];
    j = r % p.n[1];
    k = r / p.n[1];
    return p.off + (i + 1) + p.sy * (j + 1) + p.sz * (k + 1);
}
__device__ __forceinline__ int interior_index(const PatchInfo& p, int lin) {
    int i, j, k;
    return interior_cell(p, lin, i, j, k);
}

// Sums over a wavefront of NV values (a power of two): value v on the lanes of
// v * (64 / NV) ..  Each step halves the values a lane holds by trading the
// other half with its partner, so 16 values take 17 exchanges rather than 96;
// every sum adds the same pairs in the same order as wave_sum.
template <int NV>
__device__ __forceinline__ double wave_sums(const double* acc) {
    static_assert((NV & (NV - 1)) == 0 && NV <= 16, "power of two");
    const int lane = threadIdx.x & 63;
    double t[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) t[v] = acc[v];
    int o = 32;
#pragma unroll
    for (int h = NV / 2; h > 0; h /= 2, o /= 2) {
        const bool upper = lane & o;
#pragma unroll
        for (int v = 0; v < h; ++v) {
            const double keep = upper ? t[v + h] : t[v], send = upper ? t[v] : t[v + h];
            t[v] = keep + __shfl_xor(send, o, 64);
        }
    }
#pragma unroll
    for (int r = 32 / NV; r > 0; r /= 2) t[0] += __shfl_xor(t[0], r, 64);
    return t[0];
}

// Sums over a workgroup of W wavefronts of acc[0 .. nv): sum v in sh[0][v]
// after the closing barrier (one for all of them).  NV: a power of two, or one
// more.
template <int NV, int W = 4>
__device__ __forceinline__ void block_sums(double (&acc)[NV], int nv, double (*sh)[NV]) {
    constexpr int N = (NV & (NV - 1)) == 0 ? NV : NV - 1;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double s = wave_sums<N>(acc);
    if (lane % (64 / N) == 0) sh[w][lane / (64 / N)] = s;
    if (N < NV) {
        const double more = wave_sum(acc[NV - 1]);
        if (lane == 0) sh[w][NV - 1] = more;
    }
    __syncthreads();
    if ((int)threadIdx.x < nv) {
        const int v = threadIdx.x;
        double r[W];
#pragma unroll
        for (int k = 0; k < W; ++k) r[k] = sh[k][v];
#pragma unroll
        for (int n = W; n > 1; n /= 2)
#pragma unroll
            for (int k = 0; k < n / 2; ++k) r[k] = r[2 * k] + r[2 * k + 1];
        sh[0][v] = r[0];
    }
    __syncthreads();
}

// Sums of the tile partials of problem p (tiles [a, b), nv values each) into
// sh[0][v].  The loads of a step are unconditional (values beyond nv repeat the
// last one and are dropped): with a branch around each the sums waited for one
// after the other.
template <int NV, int W = 4>
__device__ __forceinline__ void partial_sums(const double* partial, int a, int b, int nv,
                                             double (*sh)[NV]) {
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    for (int i = a + threadIdx.x; i < b; i += 64 * W) {
        double x[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) x[v] = partial[(int64_t)i * nv + min(v, nv - 1)];
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += x[v];
    }
    block_sums<NV, W>(acc, nv, sh);
}

// A tile's sums (sh[0][v], after block_sums) to its partials; true in the
// workgroup that finishes its problem, to whom every partial of the problem is
// then visible.  The count is left at zero for the next launch.  Fences and
// counts are device wide (the eight XCDs have an L2 each); all stores of the
// partials are the counting wavefront's own.
__device__ __forceinline__ bool last_of_problem(const double* sums, int nv, double vol,
                                                double* partial, int32_t* count, int ntiles) {
    __shared__ int last;
    if ((int)threadIdx.x < nv) partial[(int64_t)blockIdx.x * nv + threadIdx.x] = sums[threadIdx.x] * vol;
    if (threadIdx.x < 64) {
        __threadfence();
        if (threadIdx.x == 0) {
            const int n = atomicAdd(count, 1);
            last = n == ntiles - 1;
            if (last) __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (!last) return false;
    __threadfence();
    return true;
}

// cnt (may be NULL): one zeroed counter per problem; the last tile of a
// problem then sums its partials itself and writes out[p * ostride + v]
// (NULL: k_sum_partials follows).
template <int NV>
__global__ __launch_bounds__(kBlock) void k_multidot(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ X, int64_t xs, int nv, const double* __restrict__ xsc,
    const double* __restrict__ y, double* partial, int64_t nl, int32_t* cnt,
    const int32_t* __restrict__ t0, double* out, int ostride) {
    __shared__ double sh[4][NV];
    const Tile t = vt[blockIdx.x];
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    const bool on = !active || active[t.prob];
    const PatchInfo& p = P[t.patch];
    if (on) {
        const bool cov = p.flags & PF_COVERED;
        const double sc = xsc ? xsc[t.prob] : 1.0;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            if (cov && (ctype[c] & CT_COVERED)) continue;
            const double y0 = y[c], y1 = y[c + nl];
            double x0[NV], x1[NV];                   // all loads in flight at once
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                x0[v] = X[min(v, nv - 1) * xs + c];
                x1[v] = X[min(v, nv - 1) * xs + c + nl];
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] += sc * x0[v] * y0 + sc * x1[v] * y1;
        }
    }
    block_sums<NV>(acc, nv, sh);
    if (!cnt) {
        if ((int)threadIdx.x < nv)
            partial[(int64_t)blockIdx.x * nv + threadIdx.x] = sh[0][threadIdx.x] * p.vol;
        return;
    }
    const int a = t0[t.prob], b = t0[t.prob + 1];
    if (!last_of_problem(sh[0], nv, p.vol, partial, cnt + t.prob, b - a)) return;
    partial_sums<NV>(partial, a, b, nv, sh);
    if ((int)threadIdx.x < nv) out[t.prob * ostride + threadIdx.x] = sh[0][threadIdx.x];
}

// out[p * ostride + v] = sum of the problem's tile partials (fixed order)
constexpr int kSumWaves = 16;
template <int NV>
__global__ __launch_bounds__(64 * kSumWaves) void k_sum_partials(
    const int32_t* __restrict__ t0, const double* __restrict__ partial, int nv,
    double* __restrict__ out, int ostride) {
    __shared__ double sh[kSumWaves][NV];
    const int p = blockIdx.x;
    partial_sums<NV, kSumWaves>(partial, t0[p], t0[p + 1], nv, sh);
    if ((int)threadIdx.x < nv) out[p * ostride + threadIdx.x] = sh[0][threadIdx.x];
}
static void sum_partials(const Dev& D, hipStream_t s, const double* partial, int nv, double* out,
                         int ostride) {
    auto go = [&](auto kernel) {
        kernel<<<D.nprob, 64 * kSumWaves, 0, s>>>(D.prob_vtile0, partial, nv, out, ostride);
    };
    if (nv <= 1) go(k_sum_partials<1>);
    else if (nv <= 2) go(k_sum_partials<2>);
    else if (nv <= 4) go(k_sum_partials<4>);
    else if (nv <= 8) go(k_sum_partials<8>);
    else go(k_sum_partials<16>);
}

// Launches K<NV>(args) with the smallest NV of 1, 2, 4, 8, 16 that holds nv.
#define NRD_BY_NV_T(nv, K, grid, threads, s, ...)                             \
    do {                                                                      \
        if ((nv) <= 1)                                                        \
            K<1><<<grid, threads, 0, s>>>(__VA_ARGS__);                       \
        else if ((nv) <= 2)                                                   \
            K<2><<<grid, threads, 0, s>>>(__VA_ARGS__);                       \
        else if ((nv) <= 4)                                                   \
            K<4><<<grid, threads, 0, s>>>(__VA_ARGS__);                       \
        else if ((nv) <= 8)                                                   \
            K<8><<<grid, threads, 0, s>>>(__VA_ARGS__);                       \
        else                                                                  \
            K<16><<<grid, threads, 0, s>>>(__VA_ARGS__);                      \
    } while (0)
#define NRD_BY_NV(nv, K, grid, s, ...) NRD_BY_NV_T(nv, K, grid, kBlock, s, __VA_ARGS__)

// Up to this many tiles the last workgroup of a problem sums its partials (one
// launch, 7.7 us for an inner product at 32^3 against about 10.5 us for two);
// the fence in every workgroup makes it lose beyond: 1024 tiles (128^3) 34 us
// against 17.
static int32_t* fused_count(const Dev& D) { return D.nvtiles <= kFusedTiles ? D.count : nullptr; }

void multidot(const Dev& D, hipStream_t s, const double* X, int64_t xstride, int nv,
              const double* y, double* partial, double* out, const double* xsc, bool fuse) {
    int32_t* cnt = fuse ? fused_count(D) : nullptr;
    for (int v0 = 0; v0 < nv; v0 += 16) {
        const int c = std::min(16, nv - v0);
        const double* Xc = X + v0 * xstride;
        NRD_BY_NV(c, k_multidot, D.nvtiles, s, D.vtiles, D.patches, D.ctype, D.active, Xc, xstride,
                  c, xsc, y, partial, D.nl, cnt, D.prob_vtile0, out + v0, nv);
        if (!cnt)
            sum_partials(D, s, partial, c, out + v0, nv);
    }
}

__global__ __launch_bounds__(kBlock) void k_min_pos(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ u, const double* __restrict__ du,
    const double* __restrict__ lam, double* __restrict__ partial, int64_t nl) {
    __shared__ double sh[4];
    const Tile t = vt[blockIdx.x];
    double m = DBL_MAX;
    if (!active || active[t.prob]) {
        const PatchInfo& p = P[t.patch];
        const double l = lam[t.prob];
        const bool cov = p.flags & PF_COVERED;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            if (cov && (ctype[c] & CT_COVERED)) continue;
            const double e = u[c] + l * du[c];
            const double tt = u[c + nl] + l * du[c + nl];
            // NaN compares false: map it to -1 so that it counts as a failure
            const double v = fmin(e, tt);
            m = fmin(m, (e == e && tt == tt) ? v : -1.0);
        }
    }
    const double r = block_min(m, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

__global__ __launch_bounds__(kBlock) void k_min_partials(const int32_t* __restrict__ t0,
                                                         const double* __restrict__ partial,
                                                         double* __restrict__ out) {
    __shared__ double sh[4];
    const int p = blockIdx.x;
    double m = DBL_MAX;
    for (int i = t0[p] + threadIdx.x; i < t0[p + 1]; i += kBlock) m = fmin(m, partial[i]);
    const double r = block_min(m, sh);
    if (threadIdx.x == 0) out[p] = r;
}

void min_positive(const Dev& D, hipStream_t s, const double* u, const double* du,
                  const double* lam, double* partial, double* out) {
    k_min_pos<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, u, du,
                                           lam, partial, D.nl);
    k_min_partials<<<D.nprob, kBlock, 0, s>>>(D.prob_vtile0, partial, out);
}

template <int NV>
__global__ __launch_bounds__(kBlock) void k_combine(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const int32_t* __restrict__ active, const double* __restrict__ X, int64_t xs, int nv,
    const double* __restrict__ coef, int cs, double* __restrict__ y, int accumulate,
    double alpha, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    double cf[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) cf[v] = (v < nv) ? alpha * coef[t.prob * cs + v] : 0.0;
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        double a0 = accumulate ? y[c] : 0.0;
        double a1 = accumulate ? y[c + nl] : 0.0;
        double x0[NV], x1[NV];                // all loads in flight at once
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const bool use = v < nv && cf[v] != 0.0;     // others may be stale
            x0[v] = use ? X[v * xs + c] : 0.0;
            x1[v] = use ? X[v * xs + c + nl] : 0.0;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            a0 += cf[v] * x0[v];
            a1 += cf[v] * x1[v];
        }
        y[c] = a0;
        y[c + nl] = a1;
    }
}

void combine(const Dev& D, hipStream_t s, const double* X, int64_t xstride, int nv,
             const double* coef, int cstride, double* y, int accumulate, double alpha) {
    for (int v0 = 0; v0 < nv || (v0 == 0 && nv == 0); v0 += 16) {
        const int c = std::min(16, nv - v0);
        const int acc = (v0 > 0) ? 1 : accumulate;
        const double* Xc = X + v0 * xstride;
        const double* cc = coef + v0;
        if (c <= 1)
            k_combine<1><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, Xc,
                                                      xstride, c, cc, cstride, y, acc, alpha,
                                                      D.nl);
        else if (c <= 4)
            k_combine<4><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, Xc,
                                                      xstride, c, cc, cstride, y, acc, alpha,
                                                      D.nl);
        else if (c <= 8)
            k_combine<8><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, Xc,
                                                      xstride, c, cc, cstride, y, acc, alpha,
                                                      D.nl);
        else
            k_combine<16><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, Xc,
                                                       xstride, c, cc, cstride, y, acc, alpha,
                                                       D.nl);
        if (nv == 0) break;
    }
}

// The new Hessenberg column, its Givens rotations and the residual estimate
// of one problem, by one wavefront: entry i and the rotation of row i on lane i
// (j < m <= 64), the chain of rotations in registers.  (One thread that read
// and wrote them in memory waited for each: 16 columns 10 us.)
__device__ __forceinline__ void gmres_column_one(int p, int m, int j, const double* h1,
                                                 const double* h2, double hn2,
                                                 const GmresScalars& G) {
    double* col = G.H + (int64_t)p * (m + 1) * m + (int64_t)(m + 1) * j;
    double* c = G.cs + p * m;
    double* s = G.sn + p * m;
    double* gg = G.g + p * (m + 1);
    const int lane = threadIdx.x & 63;
    const double h = lane <= j ? h1[lane] + h2[lane] : 0.0;
    const double ci = lane < j ? c[lane] : 1.0, si = lane < j ? s[lane] : 0.0;
    const double g = gg[j];
    double x = __shfl(h, 0, 64), mine = 0.0;
    for (int i = 0; i < j; ++i) {
        const double a = __shfl(ci, i, 64), b = __shfl(si, i, 64), next = __shfl(h, i + 1, 64);
        if (lane == i) mine = a * x + b * next;
        x = -b * x + a * next;
    }
    const double hn = sqrt(hn2);
    const double a = x, b = hn;
    double cc, ss, r;
    if (b == 0.0) {
        cc = 1.0;
        ss = 0.0;
        r = a;
    } else {
        r = sqrt(a * a + b * b);
        cc = a / r;
        ss = b / r;
    }
    if (lane <= j) col[lane] = lane < j ? mine : r;
    if (lane == 0) {
        c[j] = cc;
        s[j] = ss;
        col[j + 1] = 0.0;
        gg[j + 1] = -ss * g;
        gg[j] = cc * g;
        G.rho[p] = fabs(-ss * g);         // host memory, as is hn2_host
        G.hn2_host[p] = hn2;
        G.vscale[p] = hn > 0.0 ? 1.0 / hn : 0.0;
    }
}

// End of the second Gram-Schmidt pass of one problem from its sums S = (h2_0
// .. h2_j, ||w1||^2), by one wavefront: the basis is orthonormal, so w2 = w1 -
// sum h2_v v_v has ||w2||^2 = ||w1||^2 - sum h2_v^2.  Unless the second pass
// took half of it or more (w lies in the span of the basis to rounding, or is
// NaN): there the difference has lost its digits, and the column is left to the
// caller, who forms w2 and its norm (hn2_host < 0 asks for that).
__device__ __forceinline__ void gs_finish(int p, int m, int j, const double* S,
                                          const GmresScalars& G) {
    const int lane = threadIdx.x & 63;
    double n2 = S[j + 1];
    for (int v = 0; v <= j; ++v) n2 -= S[v] * S[v];
    if (lane <= j) G.h2[(int64_t)p * (j + 1) + lane] = S[lane];
    if (!(n2 >= 0.5 * S[j + 1])) {                   // uniform; NaN too
        if (lane == 0) G.hn2_host[p] = -1.0;
        return;
    }
    gmres_column_one(p, m, j, G.h1 + (int64_t)p * (j + 1), S, n2, G);
}

// Second Gram-Schmidt pass of FGMRES without storing anything: w1 = w - sum_v
// h1[p][v] v_v in registers, its inner products with the basis (h2) and its
// norm.  The corrected vector is formed only if another iteration needs it
// (k_gs_next).  Bound by reading the basis and w once, 16 (j + 2) B per cell:
// 97 us for one basis vector on an ensemble of 20 M cells (6.6 TB/s), where
// storing w1, then w2 with its norm took two passes of 155 and 187 us; 16 on 5
// M cells 196 us (338 with a branch around each vector's loads), at 32^3, where
// the sums and the new column are what takes time, 15 us (26).
template <int NV>
__global__ __launch_bounds__(kBlock) void k_gs_again(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ X, int64_t xs, int nv, const double* __restrict__ xsc,
    const double* __restrict__ w, double* partial, int64_t nl, int32_t* cnt,
    const int32_t* __restrict__ t0, int m, GmresScalars G) {
    __shared__ double sh[4][NV + 1];
    const Tile t = vt[blockIdx.x];
    double acc[NV + 1];
#pragma unroll
    for (int v = 0; v <= NV; ++v) acc[v] = 0.0;
    double nrm = 0.0;
    const bool on = !active || active[t.prob];
    const PatchInfo& p = P[t.patch];
    if (on) {
        double cf[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) cf[v] = (v < nv) ? -G.h1[t.prob * nv + v] : 0.0;
        const bool cov = p.flags & PF_COVERED;
        const double sc = xsc ? xsc[t.prob] : 1.0;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            if (cov && (ctype[c] & CT_COVERED)) continue;
            double a0 = w[c], a1 = w[c + nl];
            double x0[NV], x1[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                x0[v] = sc * X[min(v, nv - 1) * xs + c];
                x1[v] = sc * X[min(v, nv - 1) * xs + c + nl];
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {           // cf = 0 from nv on
                a0 += cf[v] * x0[v];
                a1 += cf[v] * x1[v];
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] += x0[v] * a0 + x1[v] * a1;
            nrm += a0 * a0 + a1 * a1;
        }
    }
#pragma unroll
    for (int v = 1; v <= NV; ++v)
        if (v == nv) acc[v] = nrm;
    block_sums<NV + 1>(acc, nv + 1, sh);
    if (!cnt) {
        if ((int)threadIdx.x <= nv)
            partial[(int64_t)blockIdx.x * (nv + 1) + threadIdx.x] = sh[0][threadIdx.x] * p.vol;
        return;
    }
    const int a = t0[t.prob], b = t0[t.prob + 1];
    if (!last_of_problem(sh[0], nv + 1, p.vol, partial, cnt + t.prob, b - a)) return;
    partial_sums<NV + 1>(partial, a, b, nv + 1, sh);
    if (threadIdx.x < 64 && on) gs_finish(t.prob, m, nv - 1, sh[0], G);
    if (threadIdx.x == 0 && !on) G.vscale[t.prob] = 0.0;
}

// The sums and the new column of every problem (one workgroup each).
template <int NV>
__global__ __launch_bounds__(64 * kSumWaves) void k_gs_finish(
    const int32_t* __restrict__ t0, const int32_t* __restrict__ active,
    const double* __restrict__ partial, int nv, int m, GmresScalars G) {
    __shared__ double sh[kSumWaves][NV + 1];
    const int p = blockIdx.x;
    if (active && !active[p]) {
        if (threadIdx.x == 0) G.vscale[p] = 0.0;
        return;
    }
    partial_sums<NV + 1, kSumWaves>(partial, t0[p], t0[p + 1], nv + 1, sh);
    if (threadIdx.x < 64) gs_finish(p, m, nv - 1, sh[0], G);
}

void gs_again(const Dev& D, hipStream_t s, const double* X, int64_t xstride, int nv,
              const double* w, double* partial, int m, const GmresScalars& G,
              const double* xsc) {
    int32_t* cnt = fused_count(D);
    NRD_BY_NV(nv, k_gs_again, D.nvtiles, s, D.vtiles, D.patches, D.ctype, D.active, X, xstride, nv,
              xsc, w, partial, D.nl, cnt, D.prob_vtile0, m, G);
    if (!cnt)
        NRD_BY_NV_T(nv, k_gs_finish, D.nprob, 64 * kSumWaves, s, D.prob_vtile0, D.active, partial,
                    nv, m, G);
}

// The next basis vector from the pass before: v_next = vscale (w - sum h1 v -
// sum h2 v), the corrections applied one after the other as they were found.
// With xsc (a basis of one vector read through its scale) v_0 itself is
// written too.  f (may be NULL): v_next rounded to PT, the preconditioner's
// right-hand side (colour-split where split is set), which saves the pass that
// would read v_next for it.
template <int NV, typename PT>
__global__ __launch_bounds__(kBlock) void k_gs_next(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const int32_t* __restrict__ active, double* __restrict__ X, int64_t xs, int nv,
    const double* __restrict__ r, const double* __restrict__ xsc,
    const double* __restrict__ h1, const double* __restrict__ h2,
    const double* __restrict__ w, const double* __restrict__ vscale, PT* __restrict__ f,
    int split, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    double c1[NV], c2[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        c1[v] = (v < nv) ? -h1[t.prob * nv + v] : 0.0;
        c2[v] = (v < nv) ? -h2[t.prob * nv + v] : 0.0;
    }
    const double sc = xsc ? xsc[t.prob] : 1.0, vs = vscale[t.prob];
    double* out = X + nv * xs;
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        int i, j, k;
        const int c = interior_cell(p, lin, i, j, k);
        double a0 = w[c], a1 = w[c + nl];
        double x0[NV], x1[NV];
        if (xsc) {
            x0[0] = sc * r[c];
            x1[0] = sc * r[c + nl];
            X[c] = x0[0];
            X[c + nl] = x1[0];
        } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                x0[v] = (v < nv) ? X[v * xs + c] : 0.0;
                x1[v] = (v < nv) ? X[v * xs + c + nl] : 0.0;
            }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (v < nv && c1[v] != 0.0) {
                a0 += c1[v] * x0[v];
                a1 += c1[v] * x1[v];
            }
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (v < nv && c2[v] != 0.0) {
                a0 += c2[v] * x0[v];
                a1 += c2[v] * x1[v];
            }
        a0 *= vs;
        a1 *= vs;
        out[c] = a0;
        out[c + nl] = a1;
        if (f) {
            const int cx = split ? split_index(p, i + 1, j + 1, k + 1) : c;
            f[cx] = (PT)a0;
            f[cx + nl] = (PT)a1;
        }
    }
}

template <typename PT>
void gs_next(const Dev& D, hipStream_t s, double* X, int64_t xstride, int nv, const double* r,
             const double* xsc, const double* h1, const double* h2, const double* w,
             const double* vscale, PT* f, int split) {
#define NRD_NEXT(NV)                                                                            \
    k_gs_next<NV, PT><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, X, xstride, nv, \
                                                   r, xsc, h1, h2, w, vscale, f, split, D.nl)
    if (nv <= 1)
        NRD_NEXT(1);
    else if (nv <= 2)
        NRD_NEXT(2);
    else if (nv <= 4)
        NRD_NEXT(4);
    else if (nv <= 8)
        NRD_NEXT(8);
    else
        NRD_NEXT(16);
#undef NRD_NEXT
}
template void gs_next<float>(const Dev&, hipStream_t, double*, int64_t, int, const double*,
                             const double*, const double*, const double*, const double*,
                             const double*, float*, int);
template void gs_next<double>(const Dev&, hipStream_t, double*, int64_t, int, const double*,
                              const double*, const double*, const double*, const double*,
                              const double*, double*, int);

// y -= sum_v coef[p][v] x_v (accumulating into y) and, in the same pass,
// out[p] = ||y||^2 (volume weighted over composite cells; fixed-order
// two-stage sum): the end of the second Gram-Schmidt pass of FGMRES with a
// basis of more than 16 vectors.
template <int NV>
__global__ __launch_bounds__(kBlock) void k_combine_norm(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ X, int64_t xs, int nv,
    const double* __restrict__ coef, int cs, double* __restrict__ y,
    double* __restrict__ partial, int64_t nl) {
    __shared__ double sh[4];
    const Tile t = vt[blockIdx.x];
    double acc = 0.0;
    const bool on = !active || active[t.prob];
    const PatchInfo& p = P[t.patch];
    if (on) {
        double cf[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) cf[v] = (v < nv) ? -coef[t.prob * cs + v] : 0.0;
        const bool cov = p.flags & PF_COVERED;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            double a0 = y[c], a1 = y[c + nl];
            double x0[NV], x1[NV];            // all loads in flight at once
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const bool use = v < nv && cf[v] != 0.0;
                x0[v] = use ? X[v * xs + c] : 0.0;
                x1[v] = use ? X[v * xs + c + nl] : 0.0;
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                a0 += cf[v] * x0[v];
                a1 += cf[v] * x1[v];
            }
            y[c] = a0;
            y[c + nl] = a1;
            if (!(cov && (ctype[c] & CT_COVERED))) acc += a0 * a0 + a1 * a1;
        }
    }
    const double sblk = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = sblk * p.vol;
}

void combine_norm(const Dev& D, hipStream_t s, const double* X, int64_t xstride, int nv,
                  const double* coef, int cstride, double* y, double* partial, double* out) {
    // plain combines first, the norm with the last 16
    int v0 = 0;
    for (; nv - v0 > 16; v0 += 16)
        combine(D, s, X + v0 * xstride, xstride, 16, coef + v0, cstride, y, 1, -1.0);
    const int c = nv - v0;
    NRD_BY_NV(c, k_combine_norm, D.nvtiles, s, D.vtiles, D.patches, D.ctype, D.active,
              X + v0 * xstride, xstride, c, coef + v0, cstride, y, partial, D.nl);
    sum_partials(D, s, partial, 1, out, 1);
}

// Newton update from the Krylov basis in one pass: for every active
// problem, keep = x, then x <- x - sum_v coef[p][v] z_v (the values of
// combine into s followed by axpby x <- -1 s + x), and partial = the
// minimum over the tile's composite cells of both fields of the new x (NaN
// counts as -1), as min_positive would report for the step -s.
template <int NV>
__global__ __launch_bounds__(kBlock) void k_update_min(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ Z, int64_t zs, int nv, const double* __restrict__ coef, int cs,
    double* __restrict__ x, double* __restrict__ keep, double* __restrict__ partial,
    int64_t nl) {
    __shared__ double sh[4];
    const Tile t = vt[blockIdx.x];
    double m = DBL_MAX;
    if (!active || active[t.prob]) {
        const PatchInfo& p = P[t.patch];
        double cf[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) cf[v] = (v < nv) ? coef[t.prob * cs + v] : 0.0;
        const bool cov = p.flags & PF_COVERED;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            double s0 = 0.0, s1 = 0.0;
            double z0[NV], z1[NV];            // all loads in flight at once
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const bool use = v < nv && cf[v] != 0.0;
                z0[v] = use ? Z[v * zs + c] : 0.0;
                z1[v] = use ? Z[v * zs + c + nl] : 0.0;
            }
            const double x0 = x[c], x1 = x[c + nl];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                s0 += cf[v] * z0[v];
                s1 += cf[v] * z1[v];
            }
            for (int v = NV; v < nv; ++v) {              // a basis of more than 16
                const double cv = coef[t.prob * cs + v];
                if (cv != 0.0) {
                    s0 += cv * Z[v * zs + c];
                    s1 += cv * Z[v * zs + c + nl];
                }
            }
            keep[c] = x0;
            keep[c + nl] = x1;
            const double e = -1.0 * s0 + 1.0 * x0;
            const double tt = -1.0 * s1 + 1.0 * x1;
            x[c] = e;
            x[c + nl] = tt;
            if (cov && (ctype[c] & CT_COVERED)) continue;
            m = fmin(m, (e == e && tt == tt) ? fmin(e, tt) : -1.0);
        }
    }
    const double r = block_min(m, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

void update_min(const Dev& D, hipStream_t s, const double* Z, int64_t zstride, int nv,
                const double* coef, int cstride, double* x, double* keep, double* partial,
                double* out) {
    if (nv <= 1)
        k_update_min<1><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, Z,
                                                     zstride, nv, coef, cstride, x, keep,
                                                     partial, D.nl);
    else if (nv <= 4)
        k_update_min<4><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, Z,
                                                     zstride, nv, coef, cstride, x, keep,
                                                     partial, D.nl);
    else if (nv <= 8)
        k_update_min<8><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, Z,
                                                     zstride, nv, coef, cstride, x, keep,
                                                     partial, D.nl);
    else
        k_update_min<16><<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, Z,
                                                      zstride, nv, coef, cstride, x, keep,
                                                      partial, D.nl);
    k_min_partials<<<D.nprob, kBlock, 0, s>>>(D.prob_vtile0, partial, out);
}

// Scaled max norm of the BDF2 local error estimate (eq. bdf2le):
// partial = max over the tile's composite cells of |c_p (x - x^p)| / (x + eta)
// for both fields (eta_E, eta_T), a NaN counting as infinity.
__global__ __launch_bounds__(kBlock) void k_err_max(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const int32_t* __restrict__ active,
    const double* __restrict__ x, const double* __restrict__ xp,
    const double* __restrict__ coef, double eta_E, double eta_T,
    double* __restrict__ partial, int64_t nl) {
    __shared__ double sh[4];
    const Tile t = vt[blockIdx.x];
    double m = 0.0;
    if (!active || active[t.prob]) {
        const PatchInfo& p = P[t.patch];
        const double cf = coef[t.prob];
        const bool cov = p.flags & PF_COVERED;
        for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
            const int c = interior_index(p, lin);
            if (cov && (ctype[c] & CT_COVERED)) continue;
            const double vE = fabs(cf * (x[c] - xp[c])) / (x[c] + eta_E);
            const double vT = fabs(cf * (x[c + nl] - xp[c + nl])) / (x[c + nl] + eta_T);
            const double v = fmax(vE, vT);
            m = fmax(m, (vE == vE && vT == vT) ? v : HUGE_VAL);
        }
    }
    const double r = block_max(m, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

__global__ __launch_bounds__(kBlock) void k_max_partials(const int32_t* __restrict__ t0,
                                                         const double* __restrict__ partial,
                                                         double* __restrict__ out) {
    __shared__ double sh[4];
    const int p = blockIdx.x;
    double m = 0.0;
    for (int i = t0[p] + threadIdx.x; i < t0[p + 1]; i += kBlock) m = fmax(m, partial[i]);
    const double r = block_max(m, sh);
    if (threadIdx.x == 0) out[p] = r;
}

void err_norm(const Dev& D, hipStream_t s, const double* x, const double* xp,
              const double* coef, double eta_E, double eta_T, double* partial, double* out) {
    k_err_max<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, D.active, x, xp, coef,
                                           eta_E, eta_T, partial, D.nl);
    k_max_partials<<<D.nprob, kBlock, 0, s>>>(D.prob_vtile0, partial, out);
}

__global__ __launch_bounds__(kBlock) void k_axpby(const Tile* __restrict__ vt,
                                                  const PatchInfo* __restrict__ P,
                                                  const int32_t* __restrict__ active,
                                                  const double* __restrict__ a,
                                                  const double* __restrict__ x,
                                                  const double* __restrict__ b,
                                                  double* __restrict__ y, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    const double aa = a[t.prob], bb = b[t.prob];
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        y[c] = aa * x[c] + bb * y[c];
        y[c + nl] = aa * x[c + nl] + bb * y[c + nl];
    }
}

void axpby(const Dev& D, hipStream_t s, const double* a, const double* x, const double* b,
           double* y) {
    k_axpby<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, a, x, b, y, D.nl);
}

__global__ __launch_bounds__(kBlock) void k_lincomb2(const Tile* __restrict__ vt,
                                                     const PatchInfo* __restrict__ P,
                                                     const int32_t* __restrict__ active,
                                                     const double* __restrict__ a,
                                                     const double* __restrict__ x,
                                                     const double* __restrict__ b,
                                                     const double* __restrict__ w,
                                                     double* __restrict__ y, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    const double aa = a[t.prob], bb = b[t.prob];
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        y[c] = bb * w[c] + aa * x[c];
        y[c + nl] = bb * w[c + nl] + aa * x[c + nl];
    }
}

void lincomb2(const Dev& D, hipStream_t s, const double* a, const double* x, const double* b,
              const double* w, double* y) {
    k_lincomb2<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, a, x, b, w, y, D.nl);
}

// y = u + A udot + B u_prev + C u, the terms added in that order
__global__ __launch_bounds__(kBlock) void k_bdf2_predict(const Tile* __restrict__ vt,
                                                         const PatchInfo* __restrict__ P,
                                                         const int32_t* __restrict__ active,
                                                         const double* __restrict__ cf,
                                                         const double* __restrict__ u,
                                                         const double* __restrict__ udot,
                                                         const double* __restrict__ uprev,
                                                         double* __restrict__ y,
                                                         double* __restrict__ pred,
                                                         int nprob, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    const double A = cf[t.prob], B = cf[nprob + t.prob], C = cf[2 * nprob + t.prob];
    const bool copy = A == 0.0 && B == 0.0 && C == 0.0;      // a BDF1 step: y = u
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const int64_t i = c + f * nl;
            const double uc = u[i];
            double v = uc;
            if (!copy) {
                v = A * udot[i] + v;
                v = B * uprev[i] + v;
                v = C * uc + v;
            }
            y[i] = v;
            if (pred) pred[i] = v;
        }
    }
}

void bdf2_predict(const Dev& D, hipStream_t s, const double* c, const double* u,
                  const double* udot, const double* uprev, double* y, double* pred) {
    k_bdf2_predict<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, c, u, udot,
                                                uprev, y, pred, D.nprob, D.nl);
}

__global__ __launch_bounds__(kBlock) void k_scale_copy(const Tile* __restrict__ vt,
                                                       const PatchInfo* __restrict__ P,
                                                       const int32_t* __restrict__ active,
                                                       const double* __restrict__ x,
                                                       const double* __restrict__ sc,
                                                       double* __restrict__ y, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    if (active && !active[t.prob]) return;
    const PatchInfo& p = P[t.patch];
    const double a = sc ? sc[t.prob] : 1.0;
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        y[c] = a * x[c];
        y[c + nl] = a * x[c + nl];
    }
}

void scale_copy(const Dev& D, hipStream_t s, const double* x, const double* sc, double* y) {
    k_scale_copy<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, x, sc, y, D.nl);
}
void copy_interior(const Dev& D, hipStream_t s, const double* x, double* y) {
    k_scale_copy<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.active, x, nullptr, y,
                                              D.nl);
}

// Small host arrays to the device, carried in the launch's own arguments: a
// copy from pageable memory costs the host about 15 us, this one a launch, and
// all arrays that a step of the solver needs go in one.
template <int W>
__global__ __launch_bounds__(kBlock) void k_put(const PutArgs<W> a) {
    for (int q = 0; q < a.count; ++q) {
        const PutSeg g = a.seg[q];
        for (int i = threadIdx.x; i < g.words; i += kBlock)
            g.dst[(i >> 1) * (int64_t)g.stride + (i & 1)] = a.data[g.first + i];
    }
}
void put(hipStream_t s, const PutArgs<kPutSmall>& a) { k_put<kPutSmall><<<1, kBlock, 0, s>>>(a); }
void put(hipStream_t s, const PutArgs<kPutLarge>& a) { k_put<kPutLarge><<<1, kBlock, 0, s>>>(a); }

// (n may be a whole workspace: a grid holds fewer than 2^32 threads, and a
// launch of more starts only what is left modulo 2^32, without an error)
__global__ __launch_bounds__(kBlock) void k_fill(double* __restrict__ x, int64_t n, double v) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        x[i] = v;
}
void fill_native(hipStream_t s, double* x, int64_t n, double v) {
    constexpr int64_t kMostBlocks = 1 << 16;
    const int64_t nb = (n + kBlock - 1) / kBlock;
    if (n > 0) k_fill<<<(int)std::min(nb, kMostBlocks), kBlock, 0, s>>>(x, n, v);
}

__global__ __launch_bounds__(kBlock) void k_pack(const Tile* __restrict__ vt,
                                                 const PatchInfo* __restrict__ P,
                                                 const int64_t* __restrict__ coff,
                                                 const double* __restrict__ nat,
                                                 double* __restrict__ cmp, int nf, int dir,
                                                 int64_t nl, int64_t ncells) {
    const Tile t = vt[blockIdx.x];
    const PatchInfo& p = P[t.patch];
    const int64_t base = coff[t.patch];
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        for (int f = 0; f < nf; ++f) {
            if (dir == 0)
                cmp[f * ncells + base + lin] = nat[f * nl + c];
            else
                const_cast<double*>(nat)[f * nl + c] = cmp[f * ncells + base + lin];
        }
    }
}

void pack(const Dev& D, hipStream_t s, const int64_t* coff, const double* native,
          double* compact, int nf, int64_t ncells) {
    k_pack<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, coff, native, compact, nf, 0,
                                        D.nl, ncells);
}
void unpack(const Dev& D, hipStream_t s, const int64_t* coff, const double* compact,
            double* native, int nf, int64_t ncells) {
    k_pack<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, coff, native,
                                        const_cast<double*>(compact), nf, 1, D.nl, ncells);
}

__global__ __launch_bounds__(kBlock) void k_check_pos(const Tile* __restrict__ vt,
                                                      const PatchInfo* __restrict__ P,
                                                      const double* __restrict__ x, int nf,
                                                      int32_t* __restrict__ flag,
                                                      int64_t nl) {
    const Tile t = vt[blockIdx.x];
    const PatchInfo& p = P[t.patch];
    int bad = 0;
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        for (int f = 0; f < nf; ++f) {
            const double v = x[f * nl + c];
            if (!(v > 0.0) || !(v < DBL_MAX)) bad = 1;
        }
    }
    if (bad) atomicOr(flag, 1);
}

void check_positive(const Dev& D, hipStream_t s, const double* x, int nf, int32_t* flag) {
    k_check_pos<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, x, nf, flag, D.nl);
}

__global__ __launch_bounds__(kBlock) void k_cube(const double* __restrict__ z,
                                                 double* __restrict__ z3, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const double v = z[i];
        z3[i] = v * v * v;
    }
}
void cube(hipStream_t s, const double* z, double* z3, int64_t n) {
    if (n > 0) k_cube<<<nblocks(n), kBlock, 0, s>>>(z, z3, n);
}

__global__ __launch_bounds__(kBlock) void k_to_float(const double* __restrict__ x,
                                                     float* __restrict__ y, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = (float)x[i];
}
__global__ __launch_bounds__(kBlock) void k_to_double(const float* __restrict__ x,
                                                      double* __restrict__ y, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = (double)x[i];
}
void to_float(hipStream_t s, const double* x, float* y, int64_t n) {
    if (n > 0) k_to_float<<<nblocks(n), kBlock, 0, s>>>(x, y, n);
}
void to_double(hipStream_t s, const float* x, double* y, int64_t n) {
    if (n > 0) k_to_double<<<nblocks(n), kBlock, 0, s>>>(x, y, n);
}

// ---------------------------------------------------------------------------
// Jacobian-free product (Sec. 4.1, eq. Jac-free): per-problem plain sums over
// composite cells of both fields of u.v, |v| and v.v; the differencing step
//   eps = sqrt(eps_mach) <u,v> / ||v||^2                 if |<u,v>| > u_min ||v||_1
//       = sqrt(eps_mach) u_min sign(<u,v>) ||v||_1 / ||v||^2   otherwise,
// u_min = 1e-6, sign(0) = +1, eps = 1 for v = 0; then w = u + eps v and,
// after the residual of w, Jv = (F(w) - F(u)) / eps.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_fd_sums(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const uint8_t* __restrict__ ctype, const double* __restrict__ u,
    const double* __restrict__ v, double* __restrict__ partial, int64_t nl) {
    __shared__ double sh[4];
    const Tile t = vt[blockIdx.x];
    const PatchInfo& p = P[t.patch];
    const bool cov = p.flags & PF_COVERED;
    double uv = 0.0, l1 = 0.0, v2 = 0.0;
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        if (cov && (ctype[c] & CT_COVERED)) continue;
        const double v0 = v[c], v1 = v[c + nl];
        uv += u[c] * v0 + u[c + nl] * v1;
        l1 += fabs(v0) + fabs(v1);
        v2 += v0 * v0 + v1 * v1;
    }
    uv = block_sum(uv, sh);
    l1 = block_sum(l1, sh);
    v2 = block_sum(v2, sh);
    if (threadIdx.x == 0) {
        partial[(int64_t)blockIdx.x * 3 + 0] = uv;
        partial[(int64_t)blockIdx.x * 3 + 1] = l1;
        partial[(int64_t)blockIdx.x * 3 + 2] = v2;
    }
}

__device__ __forceinline__ double fd_step(const double* __restrict__ S) {
    const double uv = S[0], l1 = S[1], v2 = S[2];
    const double root = 0x1p-26;                 // sqrt(2^-52), exact
    if (!(v2 > 0.0)) return 1.0;
    if (fabs(uv) > 1e-6 * l1) return root * uv / v2;
    const double sg = uv >= 0.0 ? 1.0 : -1.0;
    return root * 1e-6 * sg * l1 / v2;
}

__global__ __launch_bounds__(kBlock) void k_fd_shift(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const double* __restrict__ sums, const double* __restrict__ u,
    const double* __restrict__ v, double* __restrict__ w, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    const PatchInfo& p = P[t.patch];
    const double eps = fd_step(sums + 3 * t.prob);
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        w[c] = u[c] + eps * v[c];
        w[c + nl] = u[c + nl] + eps * v[c + nl];
    }
}

__global__ __launch_bounds__(kBlock) void k_fd_quotient(
    const Tile* __restrict__ vt, const PatchInfo* __restrict__ P,
    const double* __restrict__ sums, const double* __restrict__ F0,
    double* __restrict__ Jv, int64_t nl) {
    const Tile t = vt[blockIdx.x];
    const PatchInfo& p = P[t.patch];
    const double eps = fd_step(sums + 3 * t.prob);
    for (int lin = t.start + threadIdx.x; lin < t.start + t.count; lin += kBlock) {
        const int c = interior_index(p, lin);
        Jv[c] = (Jv[c] - F0[c]) / eps;
        Jv[c + nl] = (Jv[c + nl] - F0[c + nl]) / eps;
    }
}

void fd_sums(const Dev& D, hipStream_t s, const double* u, const double* v, double* partial,
             double* sums) {
    k_fd_sums<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, D.ctype, u, v, partial, D.nl);
    sum_partials(D, s, partial, 3, sums, 3);
}
void fd_shift(const Dev& D, hipStream_t s, const double* sums, const double* u,
              const double* v, double* w) {
    k_fd_shift<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, sums, u, v, w, D.nl);
}
void fd_quotient(const Dev& D, hipStream_t s, const double* sums, const double* F0,
                 double* Jv) {
    k_fd_quotient<<<D.nvtiles, kBlock, 0, s>>>(D.vtiles, D.patches, sums, F0, Jv, D.nl);
}

// ---------------------------------------------------------------------------
// FGMRES per-problem scalars (one wavefront per problem)
//   H: [nprob][(m+1) * m], column j at H[p][(m+1) j]
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(64) void k_gmres_column(int m, int j,
                                                     const int32_t* __restrict__ active,
                                                     GmresScalars G) {
    const int p = blockIdx.x;
    if (active && !active[p]) return;
    gmres_column_one(p, m, j, G.h1 + (int64_t)p * (j + 1), G.h2 + (int64_t)p * (j + 1), G.hn2[p], G);
}

void gmres_column(hipStream_t s, int nprob, int m, int j, const int32_t* active,
                  const GmresScalars& G) {
    k_gmres_column<<<nprob, 64, 0, s>>>(m, j, active, G);
}

// Back substitution by columns, row i on lane i (k <= m <= 64); eight columns
// are read at once.
__global__ __launch_bounds__(64) void k_gmres_backsolve(int m, const int32_t* __restrict__ kdim,
                                                        const double* __restrict__ H,
                                                        const double* __restrict__ g,
                                                        double* __restrict__ y) {
    const int p = blockIdx.x, lane = threadIdx.x;
    const int k = kdim[p];
    const double* Hp = H + (int64_t)p * (m + 1) * m;
    double acc = lane < k ? g[(int64_t)p * (m + 1) + lane] : 0.0, mine = 0.0;
    for (int l0 = k - 1; l0 >= 0; l0 -= 8) {
        double hc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int l = max(l0 - q, 0);
            hc[q] = lane <= l ? Hp[(m + 1) * l + lane] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int l = l0 - q;
            if (l < 0) break;                        // uniform
            const double yl = __shfl(acc, l, 64) / __shfl(hc[q], l, 64);
            if (lane == l) mine = yl;
            if (lane < l) acc -= hc[q] * yl;
        }
    }
    if (lane < m) y[(int64_t)p * m + lane] = mine;
}

void gmres_backsolve(hipStream_t s, int nprob, int m, const int32_t* kdim, const double* H,
                     const double* g, double* y) {
    k_gmres_backsolve<<<nprob, 64, 0, s>>>(m, kdim, H, g, y);
}

}  // namespace nrd

// The small grids of the base multigrid: set-up of the coarsest grid's dense
// inverse and the part of the V-cycle below a problem's tail grid, one
// workgroup per (problem, field) each (paper Sec. 4.3).
#include <hip/hip_runtime.h>

#include "pc_device.h"
#include "kernels.h"
#include "precond.h"

namespace nrd {

// ---------------------------------------------------------------------------
// numbering of the coarsest grid's cells: the longest axis slowest, so that
// neighbours lie within a half-band of N / n_max <= 25 (checked on the host)
// ---------------------------------------------------------------------------

struct BottomOrder {
    int a[3];      // axes, fastest first
    int st[3];     // stride of each (original) axis in the numbering
};

// (written with selects only, so that nothing is indexed at run time)
__device__ __forceinline__ BottomOrder bottom_order(const PatchInfo& p) {
    BottomOrder o;
    const int n0 = p.n[0], n1 = p.n[1], n2 = p.n[2];
    const int slow = (n2 > n0 && n2 > n1) ? 2 : ((n1 > n0) ? 1 : 0);
    o.a[0] = slow == 0 ? 1 : 0;
    o.a[1] = slow == 2 ? 1 : 2;
    o.a[2] = slow;
    const int na0 = slow == 0 ? n1 : n0;                  // extent of axis a[0]
    const int na1 = slow == 2 ? n1 : n2;                  // extent of axis a[1]
    o.st[0] = slow == 0 ? na0 * na1 : 1;
    o.st[1] = slow == 1 ? na0 * na1 : (slow == 0 ? 1 : na0);
    o.st[2] = slow == 2 ? na0 * na1 : na0;
    return o;
}

__device__ __forceinline__ void bottom_coords(const PatchInfo& p, const BottomOrder& o, int lin,
                                              int id[3]) {
    const int n0 = p.n[0], n1 = p.n[1], n2 = p.n[2];
    const int slow = o.a[2];
    const int na0 = slow == 0 ? n1 : n0;
    const int na1 = slow == 2 ? n1 : n2;
    const int c0 = lin % na0;
    const int r = lin / na0;
    const int c1 = r % na1;
    const int c2 = r / na1;
    // axis a[0] gets c0, a[1] gets c1, a[2] (slow) gets c2
    id[0] = slow == 0 ? c2 : c0;
    id[1] = slow == 1 ? c2 : (slow == 0 ? c0 : c1);
    id[2] = slow == 2 ? c2 : c1;
}

// floor(q / d) for 0 <= q < 2^20 and d < 2^12 from inv = 1 / d: the rounding
// of (q + 1/2) inv stays below the distance 1 / (2 d) to the next integer
// (q = 4095 and less here); an integer division costs five times as much
__device__ __forceinline__ int quot(int q, float inv) { return (int)(((float)q + 0.5f) * inv); }

// Coefficients of a coarse face (grid g of one field): the mean of the four
// fine ones.  Boundary faces included.
template <typename PT>
__device__ __forceinline__ void coarsen_field(const PatchInfo& pc, const PatchInfo& pf,
                                              const PT* Df, int64_t nlf, PT* Dc, int64_t nlc) {
    const int stc[3] = {1, pc.sy, pc.sz};
    const int stf[3] = {1, pf.sy, pf.sz};
    const float inv_x = 1.0f / (float)pc.n[0], inv_y = 1.0f / (float)pc.n[1];
    for (int lin = threadIdx.x; lin < pc.ncell; lin += blockDim.x) {
        const int r = quot(lin, inv_x), k = quot(r, inv_y);
        const int id[3] = {lin - r * pc.n[0], r - k * pc.n[1], k};
        const int c = native_index(pc, id[0], id[1], id[2]);
        const int f0 = native_index(pf, 2 * id[0], 2 * id[1], 2 * id[2]);
        // (all loads of the low faces in flight at once; few cells have others)
        PT v[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int t1 = d == 0 ? 1 : 0;
            const int t2 = d == 2 ? 1 : 2;
            const PT* src = Df + d * nlf + f0;
            v[d] = (src[0] + src[stf[t1]]) + (src[stf[t2]] + src[stf[t1] + stf[t2]]);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            Dc[d * nlc + c] = v[d] * PT(0.25);
            if (id[d] == pc.n[d] - 1) {
                const int t1 = d == 0 ? 1 : 0;
                const int t2 = d == 2 ? 1 : 2;
                const PT* src = Df + d * nlf + f0 + 2 * stf[d];
                const PT w = (src[0] + src[stf[t1]]) + (src[stf[t2]] + src[stf[t1] + stf[t2]]);
                Dc[d * nlc + c + stc[d]] = w * PT(0.25);
            }
        }
    }
}

constexpr int kSetupThreads = 1024;
static_assert(kSetupThreads == kTailThreads, "owners of the cells are the same threads");

// The inverse of the banded N x N matrix A (A(i, i - d) at [i kBottomBand + d],
// symmetric, strictly diagonally dominant) by N / 2 symmetric sweeps of two
// indices each (Gauss-Jordan, no pivoting: after the sweep of every index the
// matrix holds -A^-1).  Tiles of 4 x 4 in registers for as many threads as it
// takes; a sweep needs two columns, which their owners put into LDS, so there
// is one barrier per pair of indices and nothing else is serial.  What bounds
// it is that chain (barrier, LDS, two reciprocals) for N = 64 and the LDS reads
// for N = 125.  Cycles for N = 27, 64, 125: 14.5 k, 36.5 k, 152 k; one index at
// a time on tiles of 8 x 4, which leaves two SIMDs idle at N = 64, 23 k, 51 k,
// 146 k; pairs on 8 x 4 17 k, 39 k, 150 k.
__device__ __forceinline__ void invert(const double* A, double (*col)[2][kBottomMax], int N,
                                       double* Xi) {
    const int ld = (N + 3) >> 2, tid = threadIdx.x;
    // Wavefronts without a tile leave whole; the barriers below are passed by the
    // others alone (s_barrier waits for the wavefronts of the workgroup that have
    // not ended).
    if ((tid & ~63) >= ld * ld) return;
    const int tr = tid / ld, tc = tid - tr * ld;
    const int r0 = 4 * tr, c0 = 4 * tc;
    const bool on = tr < ld;
    double a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = r0 + i, c = c0 + j;
            const int hi = r > c ? r : c, d = r > c ? r - c : c - r;
            a[i][j] = (hi < N && d < kBottomBand) ? A[hi * kBottomBand + d] : 0.0;
        }
    // (rows and columns beyond N stay zero: their published values are zero)
    for (int kq = 0; 4 * kq < N; ++kq) {
#pragma unroll
        for (int b = 0; b < 4; b += 2) {
            const int k = 4 * kq + b;
            if (k >= N) break;                       // uniform
            // double buffered: a buffer is rewritten two barriers after it was
            // read
            double *v0 = col[b >> 1][0], *v1 = col[b >> 1][1];
            if (on && tc == kq)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v0[r0 + i] = a[i][b];
                    v1[r0 + i] = a[i][b + 1];
                }
            __syncthreads();
            if (!on) continue;
            // the inverse of the pair's 2 x 2 block (k + 1 = N: of k alone)
            const double p0 = v0[k], p1 = v0[k + 1], p2 = k + 1 < N ? v1[k + 1] : 1.0;
            double x0[4], x1[4], u0[4], u1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x0[i] = v0[r0 + i];
                x1[i] = v1[r0 + i];
                u0[i] = v0[c0 + i];
                u1[i] = v1[c0 + i];
            }
            const double i0 = rcp_nr(p0), m = p1 * i0;
            const double P11 = rcp_nr(fma(-p1, m, p2)), P01 = -m * P11, P00 = fma(-m, P01, i0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double w0 = u0[j], w1 = u1[j];
                u0[j] = fma(P00, w0, P01 * w1);
                u1[j] = fma(P01, w0, P11 * w1);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    a[i][j] = fma(-x0[i], u0[j], fma(-x1[i], u1[j], a[i][j]));
            if (tr == kq)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[b][j] = u0[j];
                    a[b + 1][j] = u1[j];
                }
            if (tc == kq) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a[i][b] = fma(P00, x0[i], P01 * x1[i]);
                    a[i][b + 1] = fma(P01, x0[i], P11 * x1[i]);
                }
                if (tr == kq) {
                    a[b][b] = -P00;
                    a[b][b + 1] = a[b + 1][b] = -P01;
                    a[b + 1][b + 1] = -P11;
                }
            }
        }
    }
    if (on)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (r0 + i < N && c0 + j < N) Xi[(r0 + i) * N + c0 + j] = -a[i][j];
}

// One grid of a tail, one field, held by the workgroup: every thread owns up
// to C cells of each colour and keeps their level operator (beta D / h^2 of
// the six faces, 0 on physical ones; the diagonal with its Marshak terms) and
// right-hand side in registers; the iterate lives in LDS, x fastest, with
// n0 n1 zeros before and after it so that no neighbour index leaves it.  Owned
// cells q: lane q & 3 of the quad of coarse cell q >> 2 owns the child with
// offsets (0,0,0), (1,1,0), (1,0,1), (0,1,1) (colour 0) and the child
// mirrored in x (colour 1).
template <typename PT, int C>
struct TailGrid {
    PT a[2][C][6], rdg[2][C], f[2][C];   // rdg: 1 / diagonal
    PT ns0[C];                           // neighbour sums colour 0 was relaxed with
    int c[2][C], nat[2][C];              // index into e (-1: no cell), native index
    int n[3], cn[3];                     // extents, extents of the next grid
    float inv_x, inv_y;                  // 1 / cn[0], 1 / cn[1]
    PT* e;

    __device__ __forceinline__ void extents(const PatchInfo& p) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            n[d] = p.n[d];
            cn[d] = p.n[d] >> 1;
        }
        inv_x = 1.0f / (float)cn[0];
        inv_y = 1.0f / (float)cn[1];
    }
    // interior coordinates of owned cell w of colour col
    __device__ __forceinline__ void place(int col, int w, int id[3]) const {
        const int q = threadIdx.x + w * kTailThreads;
        int I, J, K;
        quad_cell(q >> 2, I, J, K);
        const int lane = q & 3;
        const int child = lane == 0 ? 0 : (lane == 1 ? 3 : (lane == 2 ? 5 : 6));
        id[0] = 2 * I + ((child ^ col) & 1);
        id[1] = 2 * J + ((child >> 1) & 1);
        id[2] = 2 * K + (child >> 2);
    }
    // Set-up: the level operator of the owned cells to op, value k of colour
    // col of all cells in the order of their owners.  (Every coefficient is
    // loaded before the Marshak branch, which made each wait for the one
    // before.)
    template <typename F>
    __device__ __forceinline__ void form(const PatchInfo& p, const F& coef, double beta,
                                         int robin, PT* op) {
        extents(p);
        const int half = p.ncell >> 1;
        PT bh2[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) bh2[d] = (PT)(beta * p.ih[d] * p.ih[d]);
#pragma unroll
        for (int w = 0; w < C; ++w) {
            const int q = threadIdx.x + w * kTailThreads;
            if (q >= half) continue;
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                int id[3];
                place(col, w, id);
                PT v[6];
#pragma unroll
                for (int f = 0; f < 6; ++f) v[f] = coef(id, f);
                PT s = PT(1);
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    const int d = f >> 1;
                    const bool edge = id[d] == ((f & 1) ? n[d] - 1 : 0);
                    const PT Df = v[f];
                    v[f] = edge ? PT(0) : bh2[d] * Df;
                    s += v[f];
                    if ((robin >> f) & 1) {          // uniform
                        const PT hd = (PT)p.h[d];
                        const PT more = PT(2) * (PT)beta * Df / ((PT(4) * Df + hd) * hd);
                        s += edge ? more : PT(0);
                    }
                }
#pragma unroll
                for (int f = 0; f < 6; ++f) op[(col * 7 + f) * half + q] = v[f];
                op[(col * 7 + 6) * half + q] = PT(1) / s;
            }
        }
    }
    // the operator back into registers, and right-hand sides from ff (unless
    // NULL): loads only, in flight together with other grids'
    __device__ __forceinline__ void load(const PatchInfo& p, const PT* op,
                                         const PT* ff = nullptr) {
        extents(p);
        const int half = p.ncell >> 1;
#pragma unroll
        for (int w = 0; w < C; ++w) {
            const int q = threadIdx.x + w * kTailThreads;
            c[0][w] = c[1][w] = -1;
            if (q >= half) continue;
#pragma unroll
            for (int col = 0; col < 2; ++col) {
#pragma unroll
                for (int f = 0; f < 6; ++f) a[col][w][f] = op[(col * 7 + f) * half + q];
                rdg[col][w] = op[(col * 7 + 6) * half + q];
                int id[3];
                place(col, w, id);
                c[col][w] = id[0] + n[0] * (id[1] + n[1] * id[2]);
                nat[col][w] = native_index(p, id[0], id[1], id[2]);
                if (ff) f[col][w] = ff[nat[col][w]];
            }
        }
    }
    // e = 0 (its last reader is past a barrier)
    __device__ __forceinline__ void clear(PT* buf) {
        const int pad = n[0] * n[1];
        e = buf + pad;
        for (int q = threadIdx.x; q < n[2] * pad + 2 * pad; q += kTailThreads) buf[q] = PT(0);
    }
    __device__ __forceinline__ void quad_cell(int q, int& I, int& J, int& K) const {
        const int r = quot(q, inv_x);
        I = q - r * cn[0];
        K = quot(r, inv_y);
        J = r - K * cn[1];
    }
    __device__ __forceinline__ PT neighbours(int col, int w) const {
        const int i = c[col][w], sy = n[0], sz = n[0] * n[1];
        PT ns = PT(0);
        ns += a[col][w][0] * e[i - 1];
        ns += a[col][w][1] * e[i + 1];
        ns += a[col][w][2] * e[i - sy];
        ns += a[col][w][3] * e[i + sy];
        ns += a[col][w][4] * e[i - sz];
        ns += a[col][w][5] * e[i + sz];
        return ns;
    }
    // one colour of a red-black sweep (zero: from e = 0)
    __device__ __forceinline__ void half(int col, bool zero) {
#pragma unroll
        for (int w = 0; w < C; ++w)
            if (c[col][w] >= 0) {
                const PT ns = zero ? PT(0) : neighbours(col, w);
                e[c[col][w]] = (f[col][w] + ns) * rdg[col][w];
                if (col == 0) ns0[w] = ns;
            }
        __syncthreads();
    }
    __device__ __forceinline__ void sweeps(int nu, bool zero) {
        for (int it = 0; it < nu; ++it) {
            half(0, zero && it == 0);
            half(1, false);
        }
    }
    // fc = mean over the children of the residual.  It is zero on colour 1,
    // relaxed last; a colour-0 cell was relaxed to f + ns0 = dg e, so its
    // residual f - (dg e - ns) is what its neighbour sum has changed by since.
    __device__ __forceinline__ void restrict_to(PT* fc) const {
#pragma unroll
        for (int w = 0; w < C; ++w) {
            const int i = c[0][w];
            PT v = PT(0);
            if (i >= 0) v = neighbours(0, w) - ns0[w];
            v += __shfl_xor(v, 1);                   // quads are live or not as a whole
            v += __shfl_xor(v, 2);
            const int q = threadIdx.x + w * kTailThreads;
            if (i >= 0 && (q & 3) == 0) fc[q >> 2] = v * PT(0.125);
        }
        __syncthreads();
    }
    // e += trilinear prolongation of the next grid's ec (copy rule at edges);
    // only colour 1 unless both (the sweep that follows overwrites colour 0)
    __device__ __forceinline__ void prolong(const PT* ec, bool both) {
#pragma unroll
        for (int w = 0; w < C; ++w) {
            const int q = threadIdx.x + w * kTailThreads;
            int I, J, K;
            quad_cell(q >> 2, I, J, K);
            const int lane = q & 3;
            const int child = lane == 0 ? 0 : (lane == 1 ? 3 : (lane == 2 ? 5 : 6));
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                if (c[col][w] < 0 || (col == 0 && !both)) continue;
                const int x = min(max(I + (((child ^ col) & 1) ? 1 : -1), 0), cn[0] - 1);
                const int y = min(max(J + (((child >> 1) & 1) ? 1 : -1), 0), cn[1] - 1);
                const int z = min(max(K + ((child >> 2) ? 1 : -1), 0), cn[2] - 1);
                PT v[2][2][2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int k = 0; k < 2; ++k)
                            v[i][j][k] =
                                ec[(i ? x : I) + cn[0] * ((j ? y : J) + cn[1] * (k ? z : K))];
                e[c[col][w]] += trilinear<PT>(v);
            }
        }
        __syncthreads();
    }
};

// Set-up below a problem's tail grid: the face coefficients of the grids
// start + 1 .. depth, then the inverse X (float64, N x N, row major in the
// numbering above) of the coarsest grid's operator; in workgroups of their own
// the operators of the grids that k_mg_tail smooths.  Measured, with the
// coefficients: N = 64 (a 32^3 problem) 22.7 us, N = 125 (in an ensemble) 70
// us; a band Cholesky with two barriers per index and one triangular solve per
// column took 62 and 137 us, after two launches for the coefficients.
template <typename PT>
__global__ __launch_bounds__(kSetupThreads) void k_tail_setup(
    const int32_t* __restrict__ act, const TailEntry* __restrict__ tails, const TailGrids<PT> G,
    const ProbScalars* __restrict__ ps, double* __restrict__ X) {
    __shared__ double A[kBottomMax * kBottomBand];   // A(i, i - d) at [i kBottomBand + d]
    __shared__ __align__(16) double col[2][2][kBottomMax];
    const bool first = blockIdx.x >= (gridDim.x >> 1);      // the tail grid's own operator
    const int b = first ? blockIdx.x - (gridDim.x >> 1) : blockIdx.x;
    const TailEntry& t = tails[b >> 1];
    const int fld = b & 1;
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const int levels = t.depth - t.start;
    const int64_t na = t.grid[0].ncell, nb = levels > 1 ? t.grid[1].ncell : 0;
    PT* op = G.op + t.aoff + fld * 7 * (na + nb);
    if (first) {
        // (the second grid's coefficients as the mean of the tail grid's, the
        // expression that the other workgroup stores)
        const PatchInfo& p = t.grid[0];
        const PT* D = G.D[t.start] + fld * 3 * G.nl[t.start];
        const int64_t nl = G.nl[t.start];
        const int st[3] = {1, p.sy, p.sz};
        if (levels > 0) {
            TailGrid<PT, 2> T;
            T.form(p,
                   [&](const int id[3], int f) {
                       const int c = native_index(p, id[0], id[1], id[2]);
                       return D[(f >> 1) * nl + ((f & 1) ? c + st[f >> 1] : c)];
                   },
                   ps[t.prob].beta, fld == 0 ? p.robin : 0, op);
        }
        if (levels > 1) {
            TailGrid<PT, 1> T;
            T.form(t.grid[1],
                   [&](const int id[3], int f) {
                       const int d = f >> 1, t1 = st[d == 0 ? 1 : 0], t2 = st[d == 2 ? 1 : 2];
                       const PT* src = D + d * nl + native_index(p, 2 * id[0], 2 * id[1], 2 * id[2]) +
                                       ((f & 1) ? 2 * st[d] : 0);
                       return ((src[0] + src[t1]) + (src[t2] + src[t1 + t2])) * PT(0.25);
                   },
                   ps[t.prob].beta, fld == 0 ? t.grid[1].robin : 0, op + 7 * na);
        }
        return;
    }
    for (int g = t.start + 1; g <= t.depth; ++g) {
        const PatchInfo& pc = t.grid[g - t.start];
        const PatchInfo& pf = t.grid[g - t.start - 1];
        coarsen_field(pc, pf, G.D[g - 1] + fld * 3 * G.nl[g - 1], G.nl[g - 1],
                      G.D[g] + fld * 3 * G.nl[g], G.nl[g]);
        __threadfence_block();
        __syncthreads();
    }
    const int g = t.depth;                           // the problem's coarsest grid
    const PatchInfo& p = t.grid[g - t.start];
    const PT* D = G.D[g] + fld * 3 * G.nl[g];
    const int64_t nl = G.nl[g];
    const double beta = ps[t.prob].beta;
    // grid 0 without stored D_T: the T-field coefficients from T
    const PT* __restrict__ T0 = (g == 0 && fld == 1) ? G.T0 : nullptr;
    const PT kappa = (PT)ps[t.prob].kappa;
    const int N = p.ncell;                           // <= kBottomMax (checked on the host)
    const BottomOrder o = bottom_order(p);
    const int tid = threadIdx.x;
    for (int i = tid; i < N * kBottomBand; i += kSetupThreads) A[i] = 0.0;
    __syncthreads();
    const int st[3] = {1, p.sy, p.sz};
    for (int lin = tid; lin < N; lin += kSetupThreads) {
        int id[3];
        bottom_coords(p, o, lin, id);
        const int c = native_index(p, id[0], id[1], id[2]);
        double dg = 1.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double bh2 = beta * p.ih[d] * p.ih[d];
            const PT* Dd = D + d * nl;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (id[d] == (s ? p.n[d] - 1 : 0)) {        // grid covers the domain
                    if (fld == 0 && ((p.robin >> (2 * d + s)) & 1)) {
                        const double Dv = (double)Dd[s ? c + st[d] : c];
                        dg += 2.0 * beta * Dv / ((4.0 * Dv + p.h[d]) * p.h[d]);
                    }
                    continue;
                }
                const int nb = s ? c + st[d] : c - st[d];
                const double Dv = T0 ? (double)face_DT(T0[c], T0[nb], kappa)
                                     : (double)Dd[s ? c + st[d] : c];
                const double a = bh2 * Dv;
                dg += a;
                // the lower neighbour's entry; the upper one is that
                // neighbour's lower entry (same face, same coefficient)
                if (s == 0) A[lin * kBottomBand + o.st[d]] = -a;
            }
        }
        A[lin * kBottomBand] = dg;
    }
    __syncthreads();
    double* Xi = X + t.boff + (int64_t)fld * N * N;
    invert(A, col, N, Xi);
}

// ---------------------------------------------------------------------------
// V-cycle below the tail grid
// ---------------------------------------------------------------------------

// The V-cycle of one (problem, field) on its grids start .. depth, one
// workgroup each: the right-hand side of grid `start` is read and its
// correction written.  A grid of at most kTailCells cells is smaller than the
// launch that sweeps it, so the whole of it runs between barriers, with the
// operator in registers (as the set-up left it, in the order of its owners)
// and the iterates in LDS: a half-sweep is six LDS reads and a product per
// cell.  kTailCells is what 1024 threads hold at two cells of each colour.  The
// smallest coarsening halves 6, so two grids are smoothed at most (4096 and
// 512 cells) before the coarsest.  What bounds it is one CU's instruction rate
// and the chain of barriers; in double the registers as well (64 B per thread
// spilled).  Measured: a tail of 16^3 10.2 us in float and 18.2 in double (13.2
// and 19.3 when every cycle formed the operator from the coefficients anew, 13.9
// and 23.1 when it also waited for each of them), of the 64 problems of an
// ensemble 14.3 us, where the 13 launches it replaces took about 58 and 75 us
// in float.  A cell is relaxed by the stored reciprocal of its diagonal: a
// division here costs 2 us of a 96^3 preconditioner's 182 and leaves the cycle's
// error in single precision where it is (16^3 to 64^3 against float64: 8.04e-8 to
// 1.217e-7 either way, equal to three digits, and with one division per cell on
// every grid and no grid in one workgroup 8.07e-8 to 1.218e-7).
template <typename PT>
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(
    const int32_t* __restrict__ act, const TailEntry* __restrict__ tails, const TailGrids<PT> G,
    const double* __restrict__ X, int nu_pre, int nu_post) {
    // iterates with their padding (n0 n1 <= n / 6 where a grid coarsens)
    __shared__ PT eA[kTailCells + kTailCells / 3 + 8], eB[kTailCells / 8 + kTailCells / 24 + 8];
    __shared__ PT fB[kTailCells / 8], fC[kBottomMax], eC[kBottomMax];
    __shared__ double fv[kBottomMax];
    const TailEntry& t = tails[blockIdx.x >> 1];
    const int fld = blockIdx.x & 1;
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const int tid = threadIdx.x;
    const int levels = t.depth - t.start;            // smoothed grids (0, 1 or 2)
    const PatchInfo& pa = t.grid[0];
    const PatchInfo& pb = t.grid[1];                 // (used where levels > 1)
    const PatchInfo& pc = t.grid[levels];
    const PT* fa = G.f[t.start] + fld * G.nl[t.start];
    PT* out = G.e[t.start] + fld * G.nl[t.start];
    TailGrid<PT, 2> A;
    TailGrid<PT, 1> B;
    const int N = pc.ncell;
    const BottomOrder o = bottom_order(pc);
    int id[3] = {0, 0, 0};
    const int row = tid >> 3, part = tid & 7;        // eight lanes per row of X
    if (row < N) bottom_coords(pc, o, row, id);
    const int cell = id[0] + pc.n[0] * (id[1] + pc.n[1] * id[2]);
    const PT* op = G.op + t.aoff + (int64_t)fld * 7 * (pa.ncell + (levels > 1 ? pb.ncell : 0));
    if (levels > 0) A.load(pa, op, fa);
    // (float64: registers for one grid's operator at a time)
    constexpr bool kBoth = sizeof(PT) == 4;
    const PT* opB = op + 7 * (int64_t)pa.ncell;
    if (levels > 1) {
        if (kBoth) B.load(pb, opB);
        else B.extents(pb);
    }
    // the first 64 columns of the inverse, wanted only at the bottom (float:
    // float64 coefficients leave no registers for them)
    constexpr int kAhead = sizeof(PT) == 4 ? 8 : 0;
    const double* __restrict__ Xi = X + t.boff + (int64_t)fld * N * N;
    double xr[kAhead + 1];
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
        xr[j] = (row < N && part + 8 * j < N) ? Xi[row * N + part + 8 * j] : 0.0;
    if (levels > 0) A.clear(eA);
    if (levels > 1) B.clear(eB);
    __syncthreads();
    if (levels > 0) {
        A.sweeps(nu_pre, true);
        A.restrict_to(levels > 1 ? fB : fC);
    }
    if (levels > 1) {
        if (!kBoth) B.load(pb, opB);
#pragma unroll
        for (int col = 0; col < 2; ++col)
            if (B.c[col][0] >= 0) B.f[col][0] = fB[B.c[col][0]];
        B.sweeps(nu_pre, true);
        B.restrict_to(fC);
    }
    // coarsest grid: e = X f in float64
    if (row < N && part == 0)
        fv[row] = (double)(levels > 0 ? fC[cell] : fa[native_index(pc, id[0], id[1], id[2])]);
    __syncthreads();
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
        if (part + 8 * j < N) acc += xr[j] * fv[part + 8 * j];
    if (row < N)
        for (int j = part + 8 * kAhead; j < N; j += 8) acc += Xi[row * N + j] * fv[j];
    acc += __shfl_xor(acc, 1, 64);
    acc += __shfl_xor(acc, 2, 64);
    acc += __shfl_xor(acc, 4, 64);
    if (row < N && part == 0) {
        if (levels > 0)
            eC[cell] = (PT)acc;
        else
            out[native_index(pc, id[0], id[1], id[2])] = (PT)acc;
    }
    if (levels == 0) return;
    __syncthreads();
    if (levels > 1) {
        B.prolong(eC, nu_post == 0);
        B.sweeps(nu_post, false);
    }
    A.prolong(levels > 1 ? B.e : eC, nu_post == 0);
    A.sweeps(nu_post, false);
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            const int i = A.c[col][w];
            if (i >= 0) out[A.nat[col][w]] = A.e[i];
        }
}

// The solve of problems whose base grid does not coarsen, one workgroup per
// (problem, field).
template <typename PT>
__global__ __launch_bounds__(kBlock) void k_bottom_apply(const int32_t* __restrict__ act,
    const TailEntry* __restrict__ tails, const double* __restrict__ X, const PT* __restrict__ f, PT* __restrict__ e,
    int64_t nl, int split) {
    // split: e and f in colour-split storage
    __shared__ double fv[kBottomMax];
    const int fld = blockIdx.x & 1;
    const TailEntry& t = tails[blockIdx.x >> 1];
    if (act && !act[t.prob]) return;
    const PatchInfo& p = t.grid[0];
    const int N = p.ncell;
    const BottomOrder o = bottom_order(p);
    const double* Xi = X + t.boff + (int64_t)fld * N * N;
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
        int id[3];
        bottom_coords(p, o, j, id);
        const int c = split ? split_index(p, id[0] + 1, id[1] + 1, id[2] + 1)
                            : native_index(p, id[0], id[1], id[2]);
        fv[j] = (double)f[fld * nl + c];
    }
    __syncthreads();
    // X is symmetric: row i = column i, read with consecutive threads on
    // consecutive addresses
    for (int row = threadIdx.x; row < N; row += blockDim.x) {
        double acc = 0.0;
        for (int jj = 0; jj < N; ++jj) acc += Xi[(int64_t)jj * N + row] * fv[jj];
        int id[3];
        bottom_coords(p, o, row, id);
        const int c = split ? split_index(p, id[0] + 1, id[1] + 1, id[2] + 1)
                            : native_index(p, id[0], id[1], id[2]);
        e[fld * nl + c] = (PT)acc;
    }
}

template <typename PT>
void bottom_apply(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                  const double* X, const PT* f, PT* e, int64_t nl, int split) {
    if (n > 0) k_bottom_apply<PT><<<2 * n, kBlock, 0, s>>>(act, tails, X, f, e, nl, split);
}

template <typename PT>
void tail_setup(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                const TailGrids<PT>& G, const ProbScalars* ps, double* X) {
    if (n > 0) k_tail_setup<PT><<<4 * n, kSetupThreads, 0, s>>>(act, tails, G, ps, X);
}

template <typename PT>
void tail_cycle(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                const TailGrids<PT>& G, const double* X, int nu_pre, int nu_post) {
    if (n > 0)
        k_mg_tail<PT><<<2 * n, kTailThreads, 0, s>>>(act, tails, G, X, nu_pre, nu_post);
}

#define NRD_TAIL(PT)                                                                          \
    template void tail_setup<PT>(hipStream_t, int, const int32_t*, const TailEntry*,          \
                                 const TailGrids<PT>&, const ProbScalars*, double*);          \
    template void bottom_apply<PT>(hipStream_t, int, const int32_t*, const TailEntry*,        \
                                   const double*, const PT*, PT*, int64_t, int);              \
    template void tail_cycle<PT>(hipStream_t, int, const int32_t*, const TailEntry*,          \
                                 const TailGrids<PT>&, const double*, int, int);
NRD_TAIL(float)
NRD_TAIL(double)
#undef NRD_TAIL

}  // namespace nrd

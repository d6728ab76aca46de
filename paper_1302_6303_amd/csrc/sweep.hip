// The base grid's sweeps of the multigrid V(1,1) cycle on colour-split storage
// (problems of one level and one box), both colours in one launch each: the
// pre-sweep from zero, and the prolongation, post-sweep and coupling solve.
//
// A workgroup takes a tile of x-pairs (cells 2q, 2q + 1: one of each colour)
// and rows, one pair per thread, and marches upward in z.  Colour 1 of plane k
// needs colour 0 of planes k - 1 .. k + 1: the plane's neighbours come through
// LDS (double buffered, one barrier per plane), those above and below are the
// thread's own.  Cells on the tile's rim are relaxed by the tiles on both
// sides, so no workgroup waits for another.  Each half-sweep of its own read
// the face coefficients again, 28 B per cell and colour; here a cell's
// coefficients are formed once for both colours.  Bound by instruction issue
// and the plane's barrier (ensemble of 64 problems, 16 M cells: pre 161 us,
// post 346 us, 3 TB/s; loading a plane ahead of its use: 481 us, by its
// registers), so hierarchies whose vectors stay in the last-level cache keep
// the half-sweeps; sweep_tiles' caller has the rule.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "pc_device.h"
#include "precond.h"

namespace nrd {

// (double: its values take twice the registers, 96^3 270 against 226 us for
// the preconditioner with half-sweeps of their own)
using PT = float;

// x[i + o], i >= 0 and the offset o known or uniform: the address is a scalar
// base plus one 32-bit byte offset (a field's bytes stay below 4 GiB), half the
// address arithmetic of an index that might be negative.
__device__ __forceinline__ PT ld(const PT* x, int64_t o, uint32_t i) {
    return *reinterpret_cast<const PT*>(reinterpret_cast<const char*>(x + o) +
                                        i * (uint32_t)sizeof(PT));
}

// Level operator of the two cells of a pair at one plane: the six weights
// beta D / h^2 (0 on the domain's boundary) and the diagonal, both fields.
struct Pair {
    PT a[2][2][6];       // [cell][field][face]
    PT dg[2][2];
};

// What a thread knows of its column.
struct Column {
    int q, j, px, n1, n2, sy, sz, c, s0;     // c: native index of cell 2q, plane 0
    int robin;
    PT bh2[3], h[3], beta, kappa;
    const PT *D, *T;
    int64_t nl;
    PT zE[2], zT[2];                         // low z weights of the plane next asked for
    PT zRaw[2];                              // its low z coefficients of E

    __device__ __forceinline__ Column(const PatchInfo& p, const ProbScalars& ps, int q_, int j_,
                                      const PT* D_, const PT* T_, int64_t nl_) {
        q = q_;
        j = j_;
        px = p.n[0] >> 1;
        n1 = p.n[1];
        n2 = p.n[2];
        sy = p.sy;
        sz = p.sz;
        c = p.off + 2 * q + 1 + sy * (j + 1) + sz;
        s0 = j + p.lo[0] + p.lo[1] + p.lo[2];
        robin = p.robin;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            bh2[d] = (PT)(ps.beta * p.ih[d] * p.ih[d]);
            h[d] = (PT)p.h[d];
        }
        beta = (PT)ps.beta;
        kappa = (PT)ps.kappa;
        D = D_;
        T = T_;
        nl = nl_;
    }
    // x offset of the colour-0 cell at plane k
    __device__ __forceinline__ int zero(int k) const { return (s0 + k) & 1; }

    __device__ __forceinline__ void start(int k) {
#pragma clang fp contract(off)
        const uint32_t b = c + sz * k;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const PT Tc = ld(T, x, b), Tl = ld(T, x - sz, b);
            zRaw[x] = ld(D, 2 * nl + x, b);
            const PT wE = bh2[2] * zRaw[x], wT = bh2[2] * face_DT(Tl, Tc, kappa);
            zE[x] = k == 0 ? PT(0) : wE;
            zT[x] = k == 0 ? PT(0) : wT;
        }
    }
    // planes in order from the one given to start()
    __device__ __forceinline__ void plane(int k, Pair& P) {
#pragma clang fp contract(off)
        const uint32_t b = c + sz * k;
        const bool xl = q == 0, xh = q == px - 1, yl = j == 0, yh = j == n1 - 1, zh = k == n2 - 1;
        const PT TA = ld(T, 0, b), TB = ld(T, 1, b);
        const PT TW = ld(T, -1, b), TE = ld(T, 2, b);
        const PT TS[2] = {ld(T, -sy, b), ld(T, 1 - sy, b)},
                 TN[2] = {ld(T, sy, b), ld(T, 1 + sy, b)};
        const PT TU[2] = {ld(T, sz, b), ld(T, 1 + sz, b)};
        const PT Tc[2] = {TA, TB};
        // (every load up front and unconditional: they are all in flight at once)
        const PT DW = ld(D, 0, b), DM = ld(D, 1, b), DE = ld(D, 2, b);
        const PT DS[2] = {ld(D, nl, b), ld(D, nl + 1, b)},
                 DN[2] = {ld(D, nl + sy, b), ld(D, nl + 1 + sy, b)},
                 DU[2] = {ld(D, 2 * nl + sz, b), ld(D, 2 * nl + 1 + sz, b)};
        // x faces: west of A, between, east of B
        const PT eW = bh2[0] * DW, eM = bh2[0] * DM, eE = bh2[0] * DE;
        const PT tW = bh2[0] * face_DT(TA, TW, kappa), tM = bh2[0] * face_DT(TA, TB, kappa),
                 tE = bh2[0] * face_DT(TB, TE, kappa);
        P.a[0][0][0] = xl ? PT(0) : eW;
        P.a[0][0][1] = eM;
        P.a[1][0][0] = eM;
        P.a[1][0][1] = xh ? PT(0) : eE;
        P.a[0][1][0] = xl ? PT(0) : tW;
        P.a[0][1][1] = tM;
        P.a[1][1][0] = tM;
        P.a[1][1][1] = xh ? PT(0) : tE;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const PT sE = bh2[1] * DS[x], nE = bh2[1] * DN[x];
            const PT sT = bh2[1] * face_DT(Tc[x], TS[x], kappa),
                     nT = bh2[1] * face_DT(Tc[x], TN[x], kappa);
            P.a[x][0][2] = yl ? PT(0) : sE;
            P.a[x][0][3] = yh ? PT(0) : nE;
            P.a[x][1][2] = yl ? PT(0) : sT;
            P.a[x][1][3] = yh ? PT(0) : nT;
            const PT uE = bh2[2] * DU[x];
            const PT uT = bh2[2] * face_DT(Tc[x], TU[x], kappa);
            P.a[x][0][4] = zE[x];
            P.a[x][0][5] = zh ? PT(0) : uE;
            P.a[x][1][4] = zT[x];
            P.a[x][1][5] = zh ? PT(0) : uT;
            zE[x] = uE;
            zT[x] = uT;
#pragma unroll
            for (int fld = 0; fld < 2; ++fld) {
                PT s = PT(1);
#pragma unroll
                for (int f = 0; f < 6; ++f) s += P.a[x][fld][f];
                P.dg[x][fld] = s;
            }
        }
        // Marshak faces (bits uniform over the workgroup: usually one of six)
        auto marshak = [&](int x, int f, bool edge, PT Db) {
            if (!((robin >> f) & 1)) return;
            const PT more = robin_diag<PT>(beta, Db, h[f >> 1]);
            P.dg[x][0] += edge ? more : PT(0);
        };
        marshak(0, 0, xl, DW);
        marshak(1, 1, xh, DE);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            marshak(x, 2, yl, DS[x]);
            marshak(x, 3, yh, DN[x]);
            marshak(x, 4, k == 0, zRaw[x]);
            marshak(x, 5, zh, DU[x]);
        }
        zRaw[0] = DU[0];
        zRaw[1] = DU[1];
    }
};

// Sum of the weighted neighbours: x- x+ y- y+ z- z+.
__device__ __forceinline__ PT six(const PT a[6], PT x0, PT x1, PT y0, PT y1, PT z0, PT z1) {
    PT n = fma_t(a[0], x0, PT(0));
    n = fma_t(a[1], x1, n);
    n = fma_t(a[2], y0, n);
    n = fma_t(a[3], y1, n);
    n = fma_t(a[4], z0, n);
    return fma_t(a[5], z1, n);
}

// One colour's six weights, diagonal and right-hand side, kept for the next
// plane's iteration.
struct Held {
    PT a[2][6], dg[2], f[2];
};
__device__ __forceinline__ Held pick(const Pair& P, int x, const PT f[2]) {
    Held o;
#pragma unroll
    for (int fld = 0; fld < 2; ++fld) {
#pragma unroll
        for (int k = 0; k < 6; ++k) o.a[fld][k] = x ? P.a[1][fld][k] : P.a[0][fld][k];
        o.dg[fld] = x ? P.dg[1][fld] : P.dg[0][fld];
        o.f[fld] = f[fld];
    }
    return o;
}

// Neighbour sum of the cell at offset x of this thread's pair from the other
// colour's plane in LDS (this field's), the thread's own value of it and those
// above and below.
__device__ __forceinline__ PT around(const PT a[6], const PT* plane, int tid, int w, int x, PT own,
                                     PT below, PT above) {
    // clamped where the weight is 0 (domain edge) or the cell is not used (rim)
    const PT side = plane[x ? min(tid + 1, kSweepThreads - 1) : max(tid - 1, 0)];
    const PT south = plane[max(tid - w, 0)], north = plane[min(tid + w, kSweepThreads - 1)];
    return six(a, x ? own : side, x ? side : own, south, north, below, above);
}

// Pre-sweep from zero: colour 1 of e (colour 0 is not stored: the restriction
// reads colour 1 alone and the post-sweep relaxes colour 0 anew).  28 B per
// cell are read and written (D_E 12, T 4, f 8, e 4).
__global__ __launch_bounds__(kSweepThreads) void k_sweep_pre(
    const int32_t* __restrict__ act, const SweepTile* __restrict__ tiles,
    const PatchInfo* __restrict__ P, const ProbScalars* __restrict__ ps, const PT* __restrict__ D,
    const PT* __restrict__ T, const PT* __restrict__ f, PT* __restrict__ e, int64_t nl) {
    __shared__ PT E0[2][2][kSweepThreads];
    const SweepTile t = tiles[xcd_tile(blockIdx.x, gridDim.x)];
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const PatchInfo& p = P[t.patch];
    const int tid = threadIdx.x, w = t.w;
    const int r = tid / w;
    const bool live = r < t.nr;
    const int q = t.q0 + (live ? tid - r * w : 0), j = t.r0 + (live ? r : 0);
    const bool core = live && q >= t.cq0 && q < t.cq1 && j >= t.cr0 && j < t.cr1;
    Column col(p, ps[t.prob], q, j, D, T, nl);
    const int half = (p.sz >> 1) * (p.n[2] + 2);
    // split index of the pair's cell at offset x, plane k, colour cc
    const int sb = p.off + q + (p.sy >> 1) * (j + 1) + (p.sz >> 1);
    auto at = [&](int x, int k, int cc) { return sb + x + (p.sz >> 1) * k + cc * half; };
    const int mlo = max(t.k0 - 1, 0), mhi = min(t.k1, p.n[2] - 1);
    PT below[2] = {PT(0), PT(0)}, own[2] = {PT(0), PT(0)}, above[2];
    Held held = {};
    if (live) col.start(mlo);
    for (int m = mlo; m <= mhi + 1; ++m) {
        above[0] = above[1] = PT(0);
        Held next = {};
        if (live && m <= mhi) {
            Pair a;
            const int x0 = col.zero(m);
            const int i0 = at(x0, m, 0), i1 = at(1 - x0, m, 1);
            const PT f0[2] = {ld(f, 0, i0), ld(f, nl, i0)}, f1[2] = {ld(f, 0, i1), ld(f, nl, i1)};
            col.plane(m, a);
#pragma unroll
            for (int fld = 0; fld < 2; ++fld)
                above[fld] = relax(f0[fld], PT(0), x0 ? a.dg[1][fld] : a.dg[0][fld]);
            next = pick(a, 1 - x0, f1);
        }
        E0[m & 1][0][tid] = above[0];
        E0[m & 1][1][tid] = above[1];
        const int k = m - 1;
        if (core && k >= t.k0 && k < t.k1) {
            const int x1 = 1 - col.zero(k), i1 = at(x1, k, 1);
#pragma unroll
            for (int fld = 0; fld < 2; ++fld) {
                const PT ns = around(held.a[fld], E0[k & 1][fld], tid, w, x1, own[fld], below[fld],
                                     above[fld]);
                e[fld * nl + i1] = relax(held.f[fld], ns, held.dg[fld]);
            }
        }
        held = next;
#pragma unroll
        for (int fld = 0; fld < 2; ++fld) {
            below[fld] = own[fld];
            own[fld] = above[fld];
        }
        __syncthreads();
    }
}

// Prolongation of colour 1 (the correction of grid 1, ec), the post-sweep and,
// cell by cell, P2^-1 into y (P2: otherwise the sweep's result itself): e is
// only read.  57 B per cell are read and written (D_E 12, T 4, f 8, e 4, ec 1,
// sigma 4, z^3 8, y 16, less rims).
template <bool P2>
__global__ __launch_bounds__(kSweepThreads) void k_sweep_post(
    const int32_t* __restrict__ act, const SweepTile* __restrict__ tiles,
    const PatchInfo* __restrict__ P, const PatchInfo* __restrict__ Pc,
    const int32_t* __restrict__ cbox, const ProbScalars* __restrict__ ps,
    const PT* __restrict__ D, const PT* __restrict__ T, const PT* __restrict__ f,
    const PT* __restrict__ e, const PT* __restrict__ ec, int64_t nlc,
    const PT* __restrict__ sigma, const double* __restrict__ z3, int mode,
    double* __restrict__ y, int64_t nl) {
    __shared__ PT C1[2][2][kSweepThreads], E0[2][2][kSweepThreads];
    const SweepTile t = tiles[xcd_tile(blockIdx.x, gridDim.x)];
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const PatchInfo& p = P[t.patch];
    const PatchInfo& pc = Pc[cbox[t.prob]];
    const int tid = threadIdx.x, w = t.w;
    const int r = tid / w;
    const bool live = r < t.nr;
    const int q = t.q0 + (live ? tid - r * w : 0), j = t.r0 + (live ? r : 0);
    const bool core = live && q >= t.cq0 && q < t.cq1 && j >= t.cr0 && j < t.cr1;
    const ProbScalars& prob = ps[t.prob];
    Column col(p, prob, q, j, D, T, nl);
    const int half = (p.sz >> 1) * (p.n[2] + 2);
    const int sb = p.off + q + (p.sy >> 1) * (j + 1) + (p.sz >> 1);
    auto at = [&](int x, int k, int cc) { return sb + x + (p.sz >> 1) * k + cc * half; };
    // coarse neighbours of the pair (the base box starts at 0)
    const int cy = j >> 1, ny = min(max(cy + ((j & 1) ? 1 : -1), 0), pc.n[1] - 1);
    const int cw = max(q - 1, 0), ce = min(q + 1, pc.n[0] - 1);
    const int yc = pc.sy * (cy + 1), yn = pc.sy * (ny + 1);
    const int mlo = max(t.k0 - 2, 0), mhi = min(t.k1 + 1, p.n[2] - 1);
    const int klo = max(t.k0 - 1, 0), khi = min(t.k1, p.n[2] - 1);
    // colour 1 prolonged at planes k - 1, k, k + 1 and colour 0 relaxed at
    // planes l - 1, l, l + 1 (k = m - 1, l = m - 2)
    PT c_below[2] = {PT(0), PT(0)}, c_own[2] = {PT(0), PT(0)}, c_above[2];
    PT e_below[2] = {PT(0), PT(0)}, e_own[2] = {PT(0), PT(0)}, e_above[2];
    Held held = {};
    if (live) col.start(klo);
    for (int m = mlo; m <= mhi + 2; ++m) {
        c_above[0] = c_above[1] = PT(0);
        if (live && m <= mhi) {
            const int x1 = 1 - col.zero(m), i1 = at(x1, m, 1);
            const int cz = m >> 1, nz = min(max(cz + ((m & 1) ? 1 : -1), 0), pc.n[2] - 1);
            const int nx = x1 ? ce : cw;
            // offsets of the coarse planes (uniform) and rows
            const int64_t zo[2] = {pc.off + 1 + (int64_t)pc.sz * (cz + 1),
                                   pc.off + 1 + (int64_t)pc.sz * (nz + 1)};
#pragma unroll
            for (int fld = 0; fld < 2; ++fld) {
                const PT* s = ec + fld * nlc;
                PT v[2][2][2];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int c = 0; c < 2; ++c)
                            v[a][b][c] = ld(s, zo[c], (a ? nx : q) + (b ? yn : yc));
                c_above[fld] = ld(e, fld * nl, i1) + trilinear<PT>(v);
            }
        }
        C1[m & 1][0][tid] = c_above[0];
        C1[m & 1][1][tid] = c_above[1];
        const int k = m - 1;
        e_above[0] = e_above[1] = PT(0);
        Held next = {};
        if (live && k >= klo && k <= khi) {
            Pair a;
            const int x0 = col.zero(k);
            const int i0 = at(x0, k, 0), i1 = at(1 - x0, k, 1);
            const PT f0[2] = {ld(f, 0, i0), ld(f, nl, i0)}, f1[2] = {ld(f, 0, i1), ld(f, nl, i1)};
            col.plane(k, a);
            const Held h0 = pick(a, x0, f0);
            next = pick(a, 1 - x0, f1);
#pragma unroll
            for (int fld = 0; fld < 2; ++fld) {
                const PT ns = around(h0.a[fld], C1[k & 1][fld], tid, w, x0, c_own[fld],
                                     c_below[fld], c_above[fld]);
                e_above[fld] = relax(h0.f[fld], ns, h0.dg[fld]);
            }
        }
        E0[k & 1][0][tid] = e_above[0];
        E0[k & 1][1][tid] = e_above[1];
        const int l = m - 2;
        if (core && l >= t.k0 && l < t.k1) {
            const int x1 = 1 - col.zero(l);
            PT e1[2];
#pragma unroll
            for (int fld = 0; fld < 2; ++fld) {
                const PT ns = around(held.a[fld], E0[l & 1][fld], tid, w, x1, e_own[fld],
                                     e_below[fld], e_above[fld]);
                e1[fld] = relax(held.f[fld], ns, held.dg[fld]);
            }
            const int b = col.c + p.sz * l;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const double vE = (double)(x == x1 ? e1[0] : e_own[0]);
                const double vT = (double)(x == x1 ? e1[1] : e_own[1]);
                double yE = vE, yT = vT;
                if (P2)
                    p2_cell((double)sigma[b + x], z3[b + x], prob.beta, mode, 0, vE, vT, yE, yT);
                y[b + x] = yE;
                y[nl + b + x] = yT;
            }
        }
        held = next;
#pragma unroll
        for (int fld = 0; fld < 2; ++fld) {
            c_below[fld] = c_own[fld];
            c_own[fld] = c_above[fld];
            e_below[fld] = e_own[fld];
            e_own[fld] = e_above[fld];
        }
        __syncthreads();
    }
}

void sweep_pre(const Dev& D, hipStream_t s, const SweepTile* tiles, int nt, const PT* Dface,
               const PT* T, const PT* f, PT* e) {
    if (nt > 0)
        k_sweep_pre<<<nt, kSweepThreads, 0, s>>>(D.active, tiles, D.patches, D.ps, Dface, T, f,
                                                     e, D.nl);
}

void sweep_post(const Dev& D, hipStream_t s, const SweepTile* tiles, int nt, const PatchInfo* Pc,
                const int32_t* cbox, const PT* Dface, const PT* T, const PT* f, const PT* e,
                const PT* ec, int64_t nlc, const PT* sigma, int mode, bool p2, double* y) {
    if (nt <= 0) return;
    if (p2)
        k_sweep_post<true><<<nt, kSweepThreads, 0, s>>>(D.active, tiles, D.patches, Pc, cbox,
                                                            D.ps, Dface, T, f, e, ec, nlc, sigma,
                                                            D.z3, mode, y, D.nl);
    else
        k_sweep_post<false><<<nt, kSweepThreads, 0, s>>>(D.active, tiles, D.patches, Pc, cbox,
                                                             D.ps, Dface, T, f, e, ec, nlc, sigma,
                                                             D.z3, mode, y, D.nl);
}

// ---------------------------------------------------------------------------
// tiles
// ---------------------------------------------------------------------------

// Planes [k0, k1) of every problem's base box in runs of `chunk`; rows and
// pairs cut so that the share of threads on rims is smallest (rim: rows a
// core needs on each side; in x one pair, two cells, covers it).
static void tiles_of(const Tables& t, int rim, int chunk, std::vector<SweepTile>& out) {
    out.clear();
    for (int p = 0; p < t.nprob; ++p) {
        const int32_t b = t.level_patches[p][0][0];
        const PatchInfo& pi = t.patches[b];
        const int px = pi.n[0] >> 1, n1 = pi.n[1];
        // best cut: fewest workgroups per plane
        int bx = 0, by = 0;
        for (int nx = 1; nx <= px; ++nx) {
            const int cw = (px + nx - 1) / nx;
            const int w = std::min(px, cw + (nx > 2 ? 2 : nx - 1));
            if (w > kSweepThreads) continue;
            const int rows = kSweepThreads / w;
            int ny = 1;
            if (n1 > rows) {
                ny = 2;
                while (ny <= n1 && (n1 + ny - 1) / ny + (ny > 2 ? 2 : 1) * rim > rows) ++ny;
                if (ny > n1) continue;
            }
            if (bx == 0 || nx * ny < bx * by) {
                bx = nx;
                by = ny;
            }
        }
        const int cw = (px + bx - 1) / bx, ch = (n1 + by - 1) / by;
        for (int k0 = 0; k0 < pi.n[2]; k0 += chunk)
            for (int y = 0; y < n1; y += ch)
                for (int x = 0; x < px; x += cw) {
                    SweepTile s;
                    s.patch = b;
                    s.prob = p;
                    s.cq0 = x;
                    s.cq1 = std::min(px, x + cw);
                    s.cr0 = y;
                    s.cr1 = std::min(n1, y + ch);
                    s.q0 = std::max(0, s.cq0 - 1);
                    s.w = std::min(px, s.cq1 + 1) - s.q0;
                    s.r0 = std::max(0, s.cr0 - rim);
                    s.nr = std::min(n1, s.cr1 + rim) - s.r0;
                    s.k0 = k0;
                    s.k1 = std::min(pi.n[2], k0 + chunk);
                    out.push_back(s);
                }
    }
}

void sweep_tiles(const Tables& t, int rim, std::vector<SweepTile>& out) {
    // The longest chunk of planes that still gives every CU two workgroups
    // (a chunk repeats `rim` planes at each end), at most 16.
    for (int chunk = 16;; chunk /= 2) {
        tiles_of(t, rim, chunk, out);
        if (out.size() >= 512 || chunk == 2) return;
    }
}

}  // namespace nrd

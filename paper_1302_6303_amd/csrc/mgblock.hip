// The legs of the multigrid V(1,1) cycle on grids too large for one workgroup
// and too small to fill the chip for longer than a launch takes: everything
// between two grids in one launch each.  Down: the pre-sweep from zero and the
// restriction of its residual; up: the prolongation and the post-sweep.
//
// A workgroup takes a block of kBX x kBY x kBZ cells of one field and relaxes
// the cells around it that its own need (two rings on the first colour, one on
// the second) once more than their owners do, so nothing waits for another
// workgroup.  Iterates pass between the colours through LDS; the operator of
// every cell is loaded up front, all of it in flight at once.  Bound by launch
// and load latency: the three launches each replaces took 4 to 9 us apiece, one
// of these pays that once, for 1.9 times the relaxations.  96^3, its grids of
// 48^3 and 24^3 in blocks: preconditioner in float64 227 -> 199 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "pc_device.h"
#include "precond.h"

namespace nrd {

constexpr int kBX = 16, kBY = 8, kBZ = 8;
constexpr int kBlockThreads = 512;
constexpr int kLX = kBX + 4, kLY = kBY + 4, kLZ = kBZ + 4;     // with two rings
static_assert(kBX * kBY * kBZ == 2 * kBlockThreads, "one pair per thread");

// items of a colour in the block and `ring` rings: pairs of cells in x, one of
// each colour, row by row
constexpr int items(int ring) {
    return (ring ? kLX / 2 : kBX / 2) * (kBY + 2 * ring) * (kBZ + 2 * ring);
}
constexpr int rounds(int ring) { return (items(ring) + kBlockThreads - 1) / kBlockThreads; }

// One cell of a colour: its place in LDS (-1: none of this thread's), whether
// it lies in the domain, and its interior coordinates (clamped into it).
struct Place {
    int l, id[3];
    bool in;
};
template <int RING>
__device__ __forceinline__ Place place(const GridBlock& t, const PatchInfo& p, int item,
                                       int colour) {
    constexpr int W = RING ? kLX / 2 : kBX / 2, H = kBY + 2 * RING;
    const int row = item / W, pair = item - row * W;
    const int r = row / H;
    const int y = t.y0 - RING + row - r * H, z = t.z0 - RING + r;
    const int x = t.x0 - (RING ? 2 : 0) + 2 * pair +
                  ((colour + y + z + p.lo[0] + p.lo[1] + p.lo[2]) & 1);
    Place o;
    const bool any = item < items(RING) && x >= t.x0 - RING && x < t.x0 + kBX + RING;
    o.l = any ? (x - t.x0 + 2) + kLX * ((y - t.y0 + 2) + kLY * (z - t.z0 + 2)) : -1;
    o.in = any && x >= 0 && x < p.n[0] && y >= 0 && y < p.n[1] && z >= 0 && z < p.n[2];
    o.id[0] = min(max(x, 0), p.n[0] - 1);
    o.id[1] = min(max(y, 0), p.n[1] - 1);
    o.id[2] = min(max(z, 0), p.n[2] - 1);
    return o;
}
__device__ __forceinline__ bool inside(const GridBlock& t, const Place& o) {
    return o.in && o.id[0] >= t.x0 && o.id[0] < t.x0 + kBX && o.id[1] >= t.y0 &&
           o.id[1] < t.y0 + kBY && o.id[2] >= t.z0 && o.id[2] < t.z0 + kBZ;
}

// The operator of one field of a box that covers the domain.  SPLIT: D_T
// recomputed from T.
template <typename PT, bool SPLIT>
struct BlockOp {
    const PatchInfo& p;
    const PT *D, *T;                 // D: this field's three directions
    int64_t nl;
    PT bh2[3], beta, kappa;
    int fld;
    __device__ __forceinline__ BlockOp(const PatchInfo& p_, const ProbScalars& ps, const PT* D_,
                                       const PT* T_, int64_t nl_, int fld_)
        : p(p_), D(D_ + (int64_t)fld_ * 3 * nl_), T(T_), nl(nl_), fld(fld_) {
#pragma unroll
        for (int d = 0; d < 3; ++d) bh2[d] = (PT)(ps.beta * p.ih[d] * p.ih[d]);
        beta = (PT)ps.beta;
        kappa = (PT)ps.kappa;
    }
    // the weights beta D / h^2 of a cell's faces (0 on the boundary) and its
    // diagonal
    __device__ __forceinline__ void terms(const int id[3], PT a[6], PT& dg) const {
#pragma clang fp contract(off)
        const int c = native_index(p, id[0], id[1], id[2]);
        const int st[3] = {1, p.sy, p.sz};
        PT v[6];
        if (SPLIT && fld == 1) {                     // uniform
            const PT Tc = T[c];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                v[2 * d] = face_DT(Tc, T[c - st[d]], kappa);
                v[2 * d + 1] = face_DT(Tc, T[c + st[d]], kappa);
            }
        } else {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                v[2 * d] = D[d * nl + c];
                v[2 * d + 1] = D[d * nl + c + st[d]];
            }
        }
        dg = PT(1);
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const bool edge = id[f >> 1] == ((f & 1) ? p.n[f >> 1] - 1 : 0);
            const PT w = bh2[f >> 1] * v[f];
            a[f] = edge ? PT(0) : w;
            dg += a[f];
        }
        if (fld == 0) {                              // uniform
#pragma unroll
            for (int f = 0; f < 6; ++f)
                if ((p.robin >> f) & 1) {            // uniform
                    const bool edge = id[f >> 1] == ((f & 1) ? p.n[f >> 1] - 1 : 0);
                    const PT more = robin_diag<PT>(beta, v[f], (PT)p.h[f >> 1]);
                    dg += edge ? more : PT(0);
                }
        }
    }
    // where e and f keep a cell
    __device__ __forceinline__ int own(const int id[3]) const {
        return SPLIT ? split_index(p, id[0] + 1, id[1] + 1, id[2] + 1)
                     : native_index(p, id[0], id[1], id[2]);
    }
};

template <typename PT>
__device__ __forceinline__ PT around(const PT a[6], const PT* E, int l) {
#pragma clang fp contract(off)
    PT ns = PT(0);
    ns = fma_t(a[0], E[l - 1], ns);
    ns = fma_t(a[1], E[l + 1], ns);
    ns = fma_t(a[2], E[l - kLX], ns);
    ns = fma_t(a[3], E[l + kLX], ns);
    ns = fma_t(a[4], E[l - kLX * kLY], ns);
    return fma_t(a[5], E[l + kLX * kLY], ns);
}

// Colour 1 of e after a sweep from zero, and the next grid's right-hand side:
// the mean of the residual, which the sweep leaves at colour 0 as the sum of
// the neighbours alone (what colour 0 held is not read again, nor stored).
template <typename PT, bool SPLIT>
__global__ __launch_bounds__(kBlockThreads) void k_block_down(
    const int32_t* __restrict__ act, const GridBlock* __restrict__ blocks,
    const PatchInfo* __restrict__ P, const PatchInfo* __restrict__ Pc,
    const int32_t* __restrict__ cbox, const ProbScalars* __restrict__ ps,
    const PT* __restrict__ D, const PT* __restrict__ T, const PT* __restrict__ f,
    PT* __restrict__ e, int64_t nl, PT* __restrict__ fc, int64_t nlc) {
    __shared__ PT E[kLX * kLY * kLZ];
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const GridBlock t = blocks[b >> 1];
    const int fld = b & 1, tid = threadIdx.x;
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const PatchInfo& p = P[t.patch];
    const PatchInfo& pc = Pc[cbox[t.prob]];
    const BlockOp<PT, SPLIT> A(p, ps[t.prob], D, T, nl, fld);
    const PT* ff = f + fld * nl;
    // colour 1, one ring, and the children of a coarse cell (four lanes each)
    constexpr int N1 = rounds(1), N2 = rounds(2);
    Place q1[N1];
    PT a1[N1][6], d1[N1], f1[N1], a0[6], d0;
#pragma unroll
    for (int w = 0; w < N1; ++w) {
        q1[w] = place<1>(t, p, tid + w * kBlockThreads, 1);
        f1[w] = ff[A.own(q1[w].id)];
        A.terms(q1[w].id, a1[w], d1[w]);
    }
    const int lane = tid & 3, q = tid >> 2;
    const int child = lane == 0 ? 0 : (lane == 1 ? 3 : (lane == 2 ? 5 : 6));
    int id[3], cid[3] = {(t.x0 >> 1) + q % (kBX / 2), (t.y0 >> 1) + q / (kBX / 2) % (kBY / 2),
                         (t.z0 >> 1) + q / (kBX / 2) / (kBY / 2)};
    bool in = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int x = 2 * cid[d] + ((child >> d) & 1);
        in = in && x < p.n[d];
        id[d] = min(x, p.n[d] - 1);
    }
    A.terms(id, a0, d0);
    // colour 0 from zero, two rings
#pragma unroll
    for (int w = 0; w < N2; ++w) {
        const Place o = place<2>(t, p, tid + w * kBlockThreads, 0);
        PT a[6], dg;
        A.terms(o.id, a, dg);
        const PT v = relax(ff[A.own(o.id)], PT(0), dg);
        if (o.l >= 0) E[o.l] = o.in ? v : PT(0);
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < N1; ++w)
        if (q1[w].l >= 0) {
            const PT v = relax(f1[w], around(a1[w], E, q1[w].l), d1[w]);
            E[q1[w].l] = q1[w].in ? v : PT(0);
            if (inside(t, q1[w])) e[fld * nl + A.own(q1[w].id)] = v;
        }
    __syncthreads();
    const int l = (id[0] - t.x0 + 2) + kLX * ((id[1] - t.y0 + 2) + kLY * (id[2] - t.z0 + 2));
    PT v = in ? around(a0, E, l) : PT(0);
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    if (in && lane == 0)
        fc[fld * nlc + native_index(pc, cid[0], cid[1], cid[2])] = v * PT(0.125);
}

// out = the post-sweep from e (its colour 1) plus the prolonged ec; e is only
// read, other workgroups' rings reach into it.
template <typename PT, bool SPLIT>
__global__ __launch_bounds__(kBlockThreads) void k_block_up(
    const int32_t* __restrict__ act, const GridBlock* __restrict__ blocks,
    const PatchInfo* __restrict__ P, const PatchInfo* __restrict__ Pc,
    const int32_t* __restrict__ cbox, const ProbScalars* __restrict__ ps,
    const PT* __restrict__ D, const PT* __restrict__ T, const PT* __restrict__ f,
    const PT* __restrict__ e, int64_t nl, const PT* __restrict__ ec, int64_t nlc,
    PT* __restrict__ out) {
    __shared__ PT E[kLX * kLY * kLZ];
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const GridBlock t = blocks[b >> 1];
    const int fld = b & 1, tid = threadIdx.x;
    if (act && !act[t.prob]) return;                 // uniform over the workgroup
    const PatchInfo& p = P[t.patch];
    const PatchInfo& pc = Pc[cbox[t.prob]];
    const BlockOp<PT, SPLIT> A(p, ps[t.prob], D, T, nl, fld);
    const PT *ff = f + fld * nl, *ef = e + fld * nl, *cf = ec + fld * nlc;
    constexpr int N1 = rounds(1), N2 = rounds(2);
    // colour 0, one ring; colour 1 of the block
    Place q0[N1];
    PT a0[N1][6], d0[N1], f0[N1], a1[6], d1;
#pragma unroll
    for (int w = 0; w < N1; ++w) {
        q0[w] = place<1>(t, p, tid + w * kBlockThreads, 0);
        f0[w] = ff[A.own(q0[w].id)];
        A.terms(q0[w].id, a0[w], d0[w]);
    }
    const Place q1 = place<0>(t, p, tid, 1);
    const PT f1 = ff[A.own(q1.id)];
    A.terms(q1.id, a1, d1);
    // colour 1 prolonged, two rings
#pragma unroll
    for (int w = 0; w < N2; ++w) {
        const Place o = place<2>(t, p, tid + w * kBlockThreads, 1);
        int q[3], nb[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            q[d] = o.id[d] >> 1;
            nb[d] = min(max(q[d] + ((o.id[d] & 1) ? 1 : -1), 0), pc.n[d] - 1);
        }
        PT s[2][2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    s[i][j][k] = cf[native_index(pc, i ? nb[0] : q[0], j ? nb[1] : q[1],
                                                 k ? nb[2] : q[2])];
        const PT v = ef[A.own(o.id)] + trilinear<PT>(s);
        if (o.l >= 0) E[o.l] = o.in ? v : PT(0);
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < N1; ++w)
        if (q0[w].l >= 0) {
            const PT v = relax(f0[w], around(a0[w], E, q0[w].l), d0[w]);
            E[q0[w].l] = q0[w].in ? v : PT(0);
            if (inside(t, q0[w])) out[fld * nl + A.own(q0[w].id)] = v;
        }
    __syncthreads();
    if (q1.in) out[fld * nl + A.own(q1.id)] = relax(f1, around(a1, E, q1.l), d1);
}

template <typename PT>
void block_down(hipStream_t s, int n, const int32_t* act, const GridBlock* blocks,
                const PatchInfo* P, const PatchInfo* Pc, const int32_t* cbox,
                const ProbScalars* ps, const PT* D, const PT* T, const PT* f, PT* e, int64_t nl,
                PT* fc, int64_t nlc) {
    if (n <= 0) return;
    if (T)
        k_block_down<PT, true><<<2 * n, kBlockThreads, 0, s>>>(act, blocks, P, Pc, cbox, ps, D, T,
                                                               f, e, nl, fc, nlc);
    else
        k_block_down<PT, false><<<2 * n, kBlockThreads, 0, s>>>(act, blocks, P, Pc, cbox, ps, D,
                                                                T, f, e, nl, fc, nlc);
}

template <typename PT>
void block_up(hipStream_t s, int n, const int32_t* act, const GridBlock* blocks,
              const PatchInfo* P, const PatchInfo* Pc, const int32_t* cbox,
              const ProbScalars* ps, const PT* D, const PT* T, const PT* f, const PT* e,
              int64_t nl, const PT* ec, int64_t nlc, PT* out) {
    if (n <= 0) return;
    if (T)
        k_block_up<PT, true><<<2 * n, kBlockThreads, 0, s>>>(act, blocks, P, Pc, cbox, ps, D, T,
                                                             f, e, nl, ec, nlc, out);
    else
        k_block_up<PT, false><<<2 * n, kBlockThreads, 0, s>>>(act, blocks, P, Pc, cbox, ps, D, T,
                                                              f, e, nl, ec, nlc, out);
}

#define NRD_BLOCK(PT)                                                                           \
    template void block_down<PT>(hipStream_t, int, const int32_t*, const GridBlock*,            \
                                 const PatchInfo*, const PatchInfo*, const int32_t*,            \
                                 const ProbScalars*, const PT*, const PT*, const PT*, PT*,      \
                                 int64_t, PT*, int64_t);                                        \
    template void block_up<PT>(hipStream_t, int, const int32_t*, const GridBlock*,              \
                               const PatchInfo*, const PatchInfo*, const int32_t*,              \
                               const ProbScalars*, const PT*, const PT*, const PT*, const PT*,  \
                               int64_t, const PT*, int64_t, PT*);
NRD_BLOCK(float)
NRD_BLOCK(double)
#undef NRD_BLOCK

void grid_blocks(const PatchInfo& p, int32_t patch, int32_t prob, std::vector<GridBlock>& out) {
    for (int z = 0; z < p.n[2]; z += kBZ)
        for (int y = 0; y < p.n[1]; y += kBY)
            for (int x = 0; x < p.n[0]; x += kBX) out.push_back({patch, prob, x, y, z, {0, 0, 0}});
}

}  // namespace nrd

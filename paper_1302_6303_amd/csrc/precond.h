// Preconditioner state and drivers (see precond.hip).
#pragma once

#include "kernels.h"

namespace nrd {

constexpr int kMaxMG = 12;

// Colour-split storage of the level-0 iterate e and right-hand side f of
// the multigrid V-cycle (hierarchies whose problems have one level and one
// level-0 box, each of even x extent; `split0`).  Within the ghosted block of
// (n0 + 2)(n1 + 2)(n2 + 2) values of a box, the positions of colour 0 come
// first and those of colour 1 after them, each half in native order with
// rows of (n0 + 2) / 2 values.  The colour of ghosted position (x, y, z) is
// the parity of x + y + z + lo_0 + lo_1 + lo_2 + 1: for interior cell
// (x - 1, y - 1, z - 1) its red-black colour.  A half-sweep then reads only
// its own colour's f and the other colour's e, and writes whole lines of e.
__host__ __device__ inline int split_colour(const PatchInfo& p, int x, int y, int z) {
    return (x + y + z + p.lo[0] + p.lo[1] + p.lo[2] + 1) & 1;
}
__host__ __device__ inline int split_index(const PatchInfo& p, int x, int y, int z) {
    const int half = (p.sz >> 1) * (p.n[2] + 2);
    return p.off + split_colour(p, x, y, z) * half + (x >> 1) + (p.sy >> 1) * y +
           (p.sz >> 1) * z;
}
// Interior cell id of a box: its own split index and those of its six face
// neighbours (x-, x+, y-, y+, z-, z+; all of the other colour, so they share
// the other half's base and the neighbour's x >> 1, y and z).
__host__ __device__ inline void split_stencil(const PatchInfo& p, const int id[3], int& own,
                                              int nb[6]) {
    const int x = id[0] + 1, y = id[1] + 1, z = id[2] + 1;
    const int col = split_colour(p, x, y, z);
    const int half = (p.sz >> 1) * (p.n[2] + 2);
    const int R = p.sy >> 1, RZ = p.sz >> 1;
    const int row = R * y + RZ * z;
    own = p.off + col * half + (x >> 1) + row;
    const int ob = p.off + (1 - col) * half + row;
    nb[0] = ob + ((x - 1) >> 1);
    nb[1] = ob + ((x + 1) >> 1);
    nb[2] = ob + (x >> 1) - R;
    nb[3] = ob + (x >> 1) + R;
    nb[4] = ob + (x >> 1) - RZ;
    nb[5] = ob + (x >> 1) + RZ;
}

// Damping of the point Jacobi level smoother: 2d / (2d + 1) for d = 3, the
// weight that damps the upper half of the 7-point Laplacian's spectrum best.
constexpr double kJacobiOmega = 6.0 / 7.0;

// Coarsest grids hold at most kBottomMax cells.
constexpr int kBottomMax = 128;

// The small grids of the base multigrid (mgtail.hip).  A problem's tail
// starts at its first grid >= 1 of at most kTailCells cells; one workgroup
// per (problem, field) runs the V-cycle from there down, in LDS.
constexpr int kTailThreads = 1024;
constexpr int kTailCells = 4096;
struct TailEntry {
    int32_t prob, start, depth, pad;
    int64_t boff;            // of the problem's inverses, in doubles
    int64_t aoff;            // of the smoothed grids' operators, in values
    PatchInfo grid[3];       // grids start .. depth (at most three: each has an
                             // eighth of the cells, and 6 cells per axis or more
                             // where it coarsens)
};

// Both colours of the base grid's sweeps in one launch (sweep.hip): a tile of
// x-pairs [q0, q0 + w) and rows [r0, r0 + nr), one pair per thread, for the
// planes [k0, k1); its core [cq0, cq1) x [cr0, cr1) is written.
constexpr int kSweepThreads = 512;
constexpr int64_t kSweepLen = 8 << 20;       // least field length, ghosts included
struct SweepTile {
    int32_t patch, prob, q0, w, r0, nr, cq0, cq1, cr0, cr1, k0, k1;
};
// tiles of a hierarchy with one level-0 box per problem, even x extents, for a
// sweep whose core needs `rim` rows around it
void sweep_tiles(const Tables& t, int rim, std::vector<SweepTile>& out);
// colour 1 of e after a sweep from zero
void sweep_pre(const Dev& D, hipStream_t s, const SweepTile* tiles, int nt, const float* Dface,
               const float* T, const float* f, float* e);
// y = (p2: P2^-1 of) the sweep from e (its colour 1) plus the prolonged ec
void sweep_post(const Dev& D, hipStream_t s, const SweepTile* tiles, int nt, const PatchInfo* Pc,
                const int32_t* cbox, const float* Dface, const float* T, const float* f,
                const float* e, const float* ec, int64_t nlc, const float* sigma, int mode,
                bool p2, double* y);

// Both legs of the cycle at one grid, a launch each (mgblock.hip): blocks of a
// box that covers its problem's domain, both fields.
struct GridBlock {
    int32_t patch, prob, x0, y0, z0, pad[3];
};
constexpr int64_t kBlockCells = 1 << 20;      // largest grid in blocks, all problems
constexpr int64_t kBlockBase = 128 << 10;     // largest base grid
// a box's blocks
void grid_blocks(const PatchInfo& p, int32_t patch, int32_t prob, std::vector<GridBlock>& out);
// colour 1 of e after a sweep from zero and the coarser grid's fc (T: split
// storage of e and f, D_T from T)
template <typename PT>
void block_down(hipStream_t s, int n, const int32_t* act, const GridBlock* blocks,
                const PatchInfo* P, const PatchInfo* Pc, const int32_t* cbox,
                const ProbScalars* ps, const PT* D, const PT* T, const PT* f, PT* e, int64_t nl,
                PT* fc, int64_t nlc);
// out = the sweep from e (its colour 1) plus the prolonged ec
template <typename PT>
void block_up(hipStream_t s, int n, const int32_t* act, const GridBlock* blocks,
              const PatchInfo* P, const PatchInfo* Pc, const int32_t* cbox,
              const ProbScalars* ps, const PT* D, const PT* T, const PT* f, const PT* e,
              int64_t nl, const PT* ec, int64_t nlc, PT* out);

// Per multigrid grid: face coefficients, vectors, field length
// (kernel argument of the tail kernels).
template <typename PT>
struct TailGrids {
    PT* D[kMaxMG] = {};
    const PT* f[kMaxMG] = {};
    PT* e[kMaxMG] = {};
    int64_t nl[kMaxMG] = {};
    PT* op = nullptr;           // operators of the smoothed grids below
    const PT* T0 = nullptr;     // grid 0's T in PT when its D_T arrays are not stored
};

// coefficients below the tail grid and the coarsest grid's inverse, n problems
template <typename PT>
void tail_setup(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                const TailGrids<PT>& G, const ProbScalars* ps, double* X);
// e of grid 0 from its f for n problems whose base grid does not coarsen
template <typename PT>
void bottom_apply(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                  const double* X, const PT* f, PT* e, int64_t nl, int split);
// e of the tail grids from f of the tail grids, n problems
template <typename PT>
void tail_cycle(hipStream_t s, int n, const int32_t* act, const TailEntry* tails,
                const TailGrids<PT>& G, const double* X, int nu_pre, int nu_post);

template <typename PT>
struct PcArrays {
    const Dev* D = nullptr;
    PT* Dface = nullptr;        // 6 * nl: (field * 3 + d) * nl
    PT* sigma = nullptr;        // nl
    PT* Tp = nullptr;           // nl: T in PT (written by the snapshot when split0)
    PT* e = nullptr;            // 2 * nl each
    PT* u = nullptr;
    PT* r = nullptr;
    PT* f = nullptr;
    // per refined patch: the map of the coarse cells its prolongation reads
    const int32_t* shadow_src = nullptr;
    const ShadowPatch* shadows = nullptr;
    struct MGArr {
        int G = 0;
        const PatchInfo* box[kMaxMG] = {};
        int64_t len[kMaxMG] = {};
        const Tile* tiles[kMaxMG] = {};
        int ntiles[kMaxMG] = {};
        const int32_t* box_of[kMaxMG] = {};
        // tiles: of the problems whose grid g is their tail grid or above it;
        // smooth_tiles: of those whose grid g is above it
        const Tile* smooth_tiles[kMaxMG] = {};
        int nsmooth[kMaxMG] = {};
        int top = 0;                    // largest tail grid of any problem
        // problems whose base grid does not coarsen, then the others
        const TailEntry* tails = nullptr;
        int nbase = 0, ntail = 0;
        double* Xbuf = nullptr;
        PT* tail_op = nullptr;          // see TailGrids::op
        // first grid: per native cell, the level-0 patch of its children
        // (a base grid cut into several boxes); multi0: level 0 has siblings
        const int32_t* l0map = nullptr;
        bool multi0 = false;
        PT* Dg[kMaxMG] = {};
        PT* eg[kMaxMG] = {};
        PT* fg[kMaxMG] = {};
        // grids whose legs run in blocks (nblocks > 0), their corrections in eo
        const GridBlock* blocks[kMaxMG] = {};
        int nblocks[kMaxMG] = {};
        PT* eo[kMaxMG] = {};
        // where the correction of grid g ends up (g = 0: level 0)
        PT* result(int g) const { return nblocks[g] > 0 ? eo[g] : eg[g]; }
    } mg;
    int p2_mode = 0;
    int nu_pre = 1, nu_post = 1;
    int fac_pre = 1, fac_post = 0;   // FAC V(m, n)
    int fac_smoother = 0;            // NRD_SMOOTH_RBGS, _JACOBI or _LINE
    const Tile* ltiles = nullptr;    // x-line tiles (block Gauss-Seidel), by level
    int32_t level_line0[kMaxLev + 1] = {};
    bool base_smooth = false;        // base level: level sweeps instead of multigrid
    bool split0 = false;             // level-0 e and f in colour-split storage
    // sweep_pre / sweep_post in place of grid 0's half-sweeps
    bool fuse0 = false;
    const SweepTile *pre = nullptr, *post = nullptr;
    int npre = 0, npost = 0;
    int fac_cycle = 0;               // NRD_FAC_MULT (Alg. 1) or NRD_FAC_AFACX
    PT* e2 = nullptr;                // 2 * nl: damped Jacobi with several sweeps,
                                     // line smoother, AFACx coarse approximations
    Clock* clock = nullptr;     // times the base grid's sweeps

    void setup(hipStream_t s, const double* u_state) const;
    // y = P^-1 (wsc_p w); wsc (per problem, may be NULL) scales the input as
    // it is read
    // w NULL: input() already holds it; covered: the covered cells of y take
    // part (else they are left as the cycle leaves them)
    void apply(hipStream_t s, const double* w, double* y, const double* wsc, bool covered) const;
    // where the cycle reads its input, in PT (colour-split when split0)
    PT* input() const { return fac_cycle == NRD_FAC_AFACX ? r : f; }
    void apply_transpose(hipStream_t s, const double* w, double* y) const;
    const PT* fac(hipStream_t s, bool covered) const;    // returns u or e (one level)
    const PT* afacx(hipStream_t s, bool covered) const;  // returns e
    const PT* p1(hipStream_t s, bool covered) const;     // the configured cycle
    TailGrids<PT> tail_grids() const;
    // y (fuse0): the cycle's result goes there, through P2^-1 if p2
    void vcycle(hipStream_t s, double* y = nullptr, bool p2 = true) const;
    void composite_residual(hipStream_t s, int lev) const;
    void smooth_level(hipStream_t s, const PT* rhs, int lev, int sweeps) const;
    void correct_level(hipStream_t s, int lev, bool last) const;
    void fill_ghosts(hipStream_t s, PT* x) const;
    void restrict_(hipStream_t s, PT* x, int lev_lo) const;
    // sibling ghosts of levels lev .. lev_hi (lev_hi < 0: lev only)
    void siblings(hipStream_t s, PT* x, int lev, int lev_hi = -1) const;
    // red-black sweeps from x = 0 on A^l x = rhs over levels lo .. hi at once
    // (their patches are independent); region: only covered cells relax,
    // every other cell is set to 0
    void smooth_range(hipStream_t s, const PT* rhs, PT* x, int lo, int hi, int sweeps,
                      bool region) const;
};

}  // namespace nrd

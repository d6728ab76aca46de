"""Paths chosen by size (tiles, fused kernels), at the edges of their rules."""
import numpy as np
import pytest

from paper_1302_6303_amd import inputs as I
from tests.gpu_helpers import compact_from_native, make, native_from_compact, rel_err, to_host
from tests.helpers import state, system

pytestmark = pytest.mark.gpu


def _box(ext, seed=3):
    """One problem of the given extents with a front and two material boxes."""
    rng = np.random.default_rng(I.SEED_BASE + seed)
    prob = I.Problem(base_n=tuple(ext))
    boxes = [I.Box(0, 0, (0, 0, 0), tuple(ext))]
    z = I.eval_on_boxes(I.box_field(I.sample_material_boxes(rng, 2)), [prob], boxes)
    E, T = I.front_state([prob], boxes, rng)
    return I.Workload("box", [prob], boxes, z, E, T, np.array([1e-3]), 1)


# plane runs of 256 cells times planes: 24 (staged planes, one per tile), 1152
# (wave runs, one plane), 3456 and 8192 (wave runs, four)
@pytest.mark.parametrize("ext", [(12, 12, 24), (96, 64, 48), (96, 96, 96), (128, 128, 128)])
def test_plane_chunk_of_the_size_rule_keeps_every_value(ext):
    """The default chunk gives bit for bit the values of 16-plane chunks."""
    w = _box(ext)
    rng = np.random.default_rng(5)
    n = w.ncells()
    v = rng.standard_normal(2 * n)
    u = np.concatenate([w.compact(w.E), w.compact(w.T)]) * rng.uniform(0.9, 1.1, 2 * n)
    outs = []
    for zc in (0, 16):
        H = make(w, stencil=3, zchunk=zc, gmres_restart=2)
        H.begin_step([1e-3])
        F = H.residual(native_from_compact(H, u), H.native())
        Jv = H.jvp(native_from_compact(H, u), native_from_compact(H, v), H.native())
        outs.append((compact_from_native(H, F), compact_from_native(H, Jv)))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])


# the grid below which one workgroup runs the V-cycle (at most 4096 cells, the
# first grid or a coarser one): exactly 4096 cells, 4032 of unequal sides, one
# grid further down, the coarsest grid itself, 108 and 125 coarsest cells
@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-4)])
@pytest.mark.parametrize("ext", [(32, 32, 32), (24, 24, 56), (40, 32, 32), (8, 8, 8),
                                 (48, 48, 24), (40, 40, 40)])
def test_precond_with_small_grids_in_one_workgroup(ext, precision, tol):
    """Preconditioner against the oracle, each field normwise: operation
    order and the dense inverse in float64 (as the repository's other
    preconditioner tests), single precision of the whole cycle in mixed."""
    w = _box(ext)
    s = system(w)
    H = make(w, precision=precision, gmres_restart=2)
    H.begin_step([1e-3])
    rng = np.random.default_rng(42)
    u = state(s, w) * rng.uniform(0.9, 1.1, 2 * s.nc)
    wv = rng.standard_normal(u.shape)
    H.precond_setup(native_from_compact(H, u))
    got = compact_from_native(H, H.precond_apply(native_from_compact(H, wv), H.native()))
    ref = s.precond(u, 1e-3)[0](wv)
    for f in (slice(0, s.nc), slice(s.nc, 2 * s.nc)):
        assert rel_err(got[f], ref[f]) < tol


# reduction tiles: 256 cells each up to the size that gives 512 of them, then
# 512, 1024 and 2048; up to 256 tiles one launch sums them.  A batch: one
# counter per problem.
@pytest.mark.parametrize("exts", [[(12, 12, 12)], [(40, 40, 40)], [(48, 48, 48), (8, 8, 8)],
                                  [(64, 64, 64)], [(128, 128, 96)]])
def test_inner_products_of_every_tile_size(exts):
    """nrd_dot against exactly rounded sums (math.fsum): pairwise error of a
    tile's and the tiles' sums, well below n eps |x| |y|; twice, the counters
    of the first call reused."""
    import math
    parts = [_box(e, seed=7 + i) for i, e in enumerate(exts)]
    boxes = [I.Box(i, 0, p.boxes[0].lo, p.boxes[0].hi) for i, p in enumerate(parts)]
    w = I.Workload("dots", [p.problems[0] for p in parts], boxes, [p.z[0] for p in parts],
                   [p.E[0] for p in parts], [p.T[0] for p in parts], np.full(len(parts), 1e-3))
    H = make(w, gmres_restart=2)
    rng = np.random.default_rng(9)
    n = w.ncells()
    x, y = rng.standard_normal(2 * n), rng.standard_normal(2 * n)
    gx, gy = native_from_compact(H, x), native_from_compact(H, y)
    first = H.dot(gx, gy)
    assert H.dot(gx, gy) == first
    off = 0
    for p, (b, pr) in enumerate(zip(boxes, w.problems)):
        idx = np.r_[off:off + b.ncells, n + off:n + off + b.ncells]
        off += b.ncells
        vol = float(np.prod(pr.h()))
        prod = x[idx] * y[idx]
        ref = math.fsum(prod) * vol
        assert abs(first[p] - ref) < 1e-13 * np.abs(prod).sum() * vol


def test_newton_update_from_more_than_16_basis_vectors():
    """Steps whose Newton systems take more than 16 Krylov vectors in one
    cycle: every vector enters the update, so the iteration counts follow
    those of a basis of 16 with restarts (both solve each system to the same
    forcing tolerance: at most one Newton iteration apart)."""
    w = I.marshak_single(32, state="front")
    st = []
    for m in (64, 16):
        H = make(w, gmres_restart=m, gmres_maxrestarts=60, bdf_max_order=1, fac_base=1)
        st.append(H.implicit_step([6e-3])[1][0])
    assert max(st[0]["krylov_per_newton"]) > 16
    assert abs(st[0]["newton_iters"] - st[1]["newton_iters"]) <= 1


@pytest.mark.parametrize("precision", [0, 1])
def test_gradient_with_a_long_krylov_basis(precision):
    """Transposed solves to 1e-12 with a weak preconditioner: a basis of 64
    (more than 16 vectors take the in-place passes) and one of 16 with
    restarts solve the same systems, which the gradient keeps to 1e-9."""
    w = I.marshak_single(16, state="front")
    out = []
    for m in (64, 16):
        H = make(w, precision=precision, gmres_restart=m, gmres_maxrestarts=60, bdf_max_order=1,
                 adjoint_slots=6, fac_base=1)
        out.append(to_host(H.adjoint_run([2e-3], 1, 1)))
    assert rel_err(out[0], out[1]) < 1e-9


# one launch per base-grid sweep from 8 M cells on: the first (a filler)
# brings the hierarchy above; pairs and rows cut or not, three pairs only,
# fewer planes than a run of 16, runs with a remainder
SWEEP_EXTS = [(256, 256, 192), (10, 14, 6), (6, 8, 10), (128, 64, 64), (48, 80, 48),
              (20, 12, 20), (192, 96, 96), (14, 6, 10), (80, 80, 80)]


def _sweep_batch():
    """The problems of SWEEP_EXTS, Marshak faces in turn on every side, and
    one hierarchy of them all."""
    ws = [_box(e, seed=30 + i) for i, e in enumerate(SWEEP_EXTS)]
    for p, w in enumerate(ws):
        w.problems[0].bc_E = tuple(int((f + p) % 3 == 0) for f in range(6))
        w.dt = np.array([2e-5 / (1 + p)])
    boxes = [I.Box(p, 0, (0, 0, 0), e) for p, e in enumerate(SWEEP_EXTS)]
    return ws, I.Workload("several", [x.problems[0] for x in ws], boxes, [x.z[0] for x in ws],
                          [x.E[0] for x in ws], [x.T[0] for x in ws],
                          np.concatenate([x.dt for x in ws]))


def test_base_sweeps_in_one_launch_keep_every_value():
    """Each problem's preconditioner beside the others, and alone in a small
    hierarchy (a launch per colour): bit for bit the same, as both form every
    value by the same operations."""
    ws, w = _sweep_batch()
    n = [x.ncells() for x in ws]
    us = [np.concatenate([x.compact(x.E), x.compact(x.T)]) for x in ws]
    vs = [np.random.default_rng(60 + p).standard_normal(2 * n[p]) for p in range(len(ws))]

    def apply(w, u, v):
        H = make(w, precision=1, gmres_restart=2)
        H.begin_step([float(x) for x in w.dt])
        H.precond_setup(native_from_compact(H, u))
        return compact_from_native(H, H.precond_apply(native_from_compact(H, v), H.native()))

    def join(xs):                        # every E field, then every T field
        return np.concatenate([x[:k] for x, k in zip(xs, n)] + [x[k:] for x, k in zip(xs, n)])

    got = apply(w, join(us), join(vs))
    at = np.concatenate([[0], np.cumsum(n)])
    for p in range(1, len(ws)):
        want = apply(ws[p], us[p], vs[p])
        mine = np.concatenate([got[f + at[p]:f + at[p + 1]] for f in (0, at[-1])])
        np.testing.assert_array_equal(mine, want, err_msg=str(SWEEP_EXTS[p]))


def test_gradient_through_the_base_sweeps_in_one_launch():
    """The transposed cycle (no coupling solve in its last launch): gradient
    of each problem beside the others and alone.  The systems are the same
    and solved to 1e-12; inner products are summed in other groups."""
    ws, w = _sweep_batch()
    opt = dict(precision=1, gmres_restart=16, bdf_max_order=1, adjoint_slots=6)
    got = to_host(make(w, **opt).adjoint_run([float(x) for x in w.dt], 1, 1))
    at = np.concatenate([[0], np.cumsum([x.ncells() for x in ws])])
    for p in range(1, len(ws)):
        want = to_host(make(ws[p], **opt).adjoint_run([float(ws[p].dt[0])], 1, 1))
        assert rel_err(got[at[p]:at[p + 1]], want) < 1e-9, SWEEP_EXTS[p]


def _grid(base, fine):
    """Problems of the given base extents (equal ones share their fields) and
    refined boxes (lo, hi) of the first."""
    rng = np.random.default_rng(I.SEED_BASE + 70)
    problems, boxes = [], []
    for p, e in enumerate(base):
        problems.append(I.Problem(base_n=tuple(e), bc_E=(1, 0, 1, 1, 0, 1)))
        boxes.append(I.Box(p, 0, (0, 0, 0), tuple(e)))
    boxes += [I.Box(0, 1, lo, hi) for lo, hi in fine]
    z = I.eval_on_boxes(I.box_field(I.sample_material_boxes(rng, 2)), problems, boxes)
    E, T = I.front_state(problems, boxes, rng)
    return I.Workload("grid", problems, boxes, z, E, T, np.full(len(base), 1e-3))


# staged planes / wave runs: one-plane tiles 8 and 192 | 200, 12000 | 12008;
# rows of 20 and 8 cells (with their ghost a whole share of a wavefront's 63
# entries); wide rows; refined boxes of 60, 62, 126, 128 and 256 cells in x
FINE = [((0, 0, 0), (126, 10, 40)), ((0, 20, 0), (62, 30, 40)), ((64, 20, 2), (124, 32, 42)),
        ((0, 40, 60), (128, 46, 90))]


@pytest.mark.parametrize("base,fine", [
    ([(8, 8, 8)], []), ([(8, 8, 8)] * 24, []), ([(8, 8, 8)] * 25, []), ([(80, 80, 80)] * 6, []),
    ([(80, 80, 80)] * 6 + [(8, 8, 8)], []), ([(20, 12, 20)] * 12, []), ([(128, 64, 64)], []),
    ([(64, 64, 64)], FINE), ([(128, 64, 64)], [((0, 0, 0), (256, 8, 24))])])
def test_stencil_kernel_of_the_size_rule(base, fine):
    """Residual and Jacobian action by the default kernel against one thread
    per cell: the same formulas of every face and cell, fused differently
    kernel by kernel.  Rounding of a face's chain of about twenty operations,
    of seven faces and terms: a few hundred ulp of the largest at most."""
    w = _grid(base, fine)
    rng = np.random.default_rng(5)
    n = w.ncells()
    v = rng.standard_normal(2 * n)
    u = np.concatenate([w.compact(w.E), w.compact(w.T)]) * rng.uniform(0.9, 1.1, 2 * n)
    outs = []
    for st in (3, 0):
        H = make(w, stencil=st, gmres_restart=2)
        H.begin_step([float(x) for x in w.dt])
        F = H.residual(native_from_compact(H, u), H.native())
        Jv = H.jvp(native_from_compact(H, u), native_from_compact(H, v), H.native())
        outs.append((compact_from_native(H, F), compact_from_native(H, Jv)))
    for got, ref in zip(*outs):
        assert rel_err(got, ref) < 1e-13


# grids whose legs of the cycle run in blocks of 16 x 8 x 8 cells: base grid 6
# cells wide (one clipped block), whole blocks, remainders in every direction,
# 110 592 cells (the largest cube), 184 320 (the base grid in half-sweeps, the
# next in blocks)
BLOCK_EXTS = [(6, 8, 10), (10, 14, 6), (20, 12, 20), (32, 32, 32), (40, 40, 40), (24, 24, 40),
              (24, 40, 40), (40, 24, 24), (48, 48, 48), (48, 80, 48)]


@pytest.mark.parametrize("precision", [1, 0])
def test_cycle_legs_in_blocks_keep_every_value(precision):
    """Each problem's preconditioner alone (blocks where the grid is small)
    and beside a filler that brings its first two grids above the rule (other
    kernels): bit for bit the same."""
    fill = (192, 256, 192)
    ws = [_box(e, seed=80 + i) for i, e in enumerate([fill] + BLOCK_EXTS)]
    for p, w in enumerate(ws):
        w.problems[0].bc_E = tuple(int((f + p) % 3 == 0) for f in range(6))
    w = I.Workload("several", [x.problems[0] for x in ws],
                   [I.Box(p, 0, (0, 0, 0), e) for p, e in enumerate([fill] + BLOCK_EXTS)],
                   [x.z[0] for x in ws], [x.E[0] for x in ws], [x.T[0] for x in ws],
                   np.array([2e-5 / (1 + p) for p in range(len(ws))]))
    n = [x.ncells() for x in ws]
    us = [np.concatenate([x.compact(x.E), x.compact(x.T)]) for x in ws]
    vs = [np.random.default_rng(90 + p).standard_normal(2 * n[p]) for p in range(len(ws))]

    def apply(w, dt, u, v):
        H = make(w, precision=precision, gmres_restart=2)
        H.begin_step(dt)
        H.precond_setup(native_from_compact(H, u))
        return compact_from_native(H, H.precond_apply(native_from_compact(H, v), H.native()))

    def join(xs):
        return np.concatenate([x[:k] for x, k in zip(xs, n)] + [x[k:] for x, k in zip(xs, n)])

    got = apply(w, [float(x) for x in w.dt], join(us), join(vs))
    at = np.concatenate([[0], np.cumsum(n)])
    for p in range(1, len(ws)):
        want = apply(ws[p], [float(w.dt[p])], us[p], vs[p])
        mine = np.concatenate([got[f + at[p]:f + at[p + 1]] for f in (0, at[-1])])
        np.testing.assert_array_equal(mine, want, err_msg=str(BLOCK_EXTS[p - 1]))


@pytest.mark.parametrize("m", [1, 5, 8, 9, 33])
def test_gradient_with_a_basis_of_any_size(m):
    """Columns, rotations and back substitution of 1 to 33 vectors (whole and
    partly used groups of 1, 2, 4, 8 and 16).  The transposed systems are
    solved to 1e-12 and the step they belong to to 1e-12 of its first
    residual (the default 1e-8 leaves states 1e-10 and gradients 6e-9 apart),
    which the gradient keeps to 1e-9.  One vector: with the multigrid
    preconditioner, which needs few."""
    w = I.marshak_single(16, state="front")
    out = []
    for k in (64, m):
        H = make(w, precision=0, gmres_restart=k, gmres_maxrestarts=400, bdf_max_order=1,
                 adjoint_slots=6, newton_rtol=1e-12, fac_base=int(m > 1))
        out.append(to_host(H.adjoint_run([2e-3], 1, 1)))
    assert rel_err(out[0], out[1]) < 1e-9


@pytest.mark.parametrize("ext", [(3, 1, 1), (2, 2, 1), (5, 3, 2), (12, 12, 12), (10, 14, 6), (6, 8, 10),
                                 (5, 5, 5)])
def test_coarsest_grids_of_any_size(ext):
    """The dense inverse of 3, 4, 30 and 125 cells (base grids that do not
    coarsen) and of 27, 105 and 60: odd counts end on a single index, tiles
    of four on a remainder of each size.  Tolerance as above."""
    test_precond_with_small_grids_in_one_workgroup(ext, 0, 1e-10)


def test_gathers_of_the_transpose_take_any_row_length():
    """Coarse sources of a transposed product gather their ghosts' values four
    at a time: <lam, J v> = <J^T lam, v> on a hierarchy of three levels whose
    sources feed 1 to many ghosts, to the rounding of sums of n products."""
    w = I.static_amr(base=16, nlevels=3, side=(4, 12), seed_k=12, state="front")
    H = make(w, gmres_restart=2)
    H.begin_step([1e-3])
    rng = np.random.default_rng(3)
    n = w.ncells()
    u = np.concatenate([w.compact(w.E), w.compact(w.T)]) * rng.uniform(0.9, 1.1, 2 * n)
    un = native_from_compact(H, u)
    v, lam = (rng.standard_normal(2 * n) for _ in range(2))
    # (both arguments on composite cells alone: the product's first step makes
    # covered ones the mean of their children)
    Jv = compact_from_native(H, H.jvp(un, native_from_compact(H, v), H.native()))
    lam[Jv == 0.0] = 0.0
    v0 = v.copy()
    Jt = compact_from_native(H, H.vjp(un, native_from_compact(H, lam), H.native())[0])
    a, b = float(lam @ Jv), float(Jt @ v0)
    assert abs(a - b) < 1e-12 * float(np.abs(lam) @ np.abs(Jv) + np.abs(Jt) @ np.abs(v0))

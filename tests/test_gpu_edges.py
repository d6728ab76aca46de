"""Edges of the solver's ranges: overflow and NaN, cycles other than V(1,1),
hundreds of problems, the tile tuner's cache."""
import time

import numpy as np
import pytest
import torch

from oracle import precond as pc
from paper_1302_6303_amd import inputs as I
from tests.gpu_helpers import (compact_from_native, make, native_from_compact, problem_slices,
                               rel_err)
from tests.helpers import state, system
from tests.test_gpu_paths import _box, _grid, _sweep_batch
from tests.test_gpu_paths import test_stencil_kernel_of_the_size_rule as _one_kernel

pytestmark = pytest.mark.gpu


def _uniform(ext, kappa, E=1.0, T=1.0):
    """One problem with E, T and z = 1 the same in every cell."""
    w = _box(ext)
    w.problems[0].kappa = kappa
    w.E, w.T, w.z = ([np.full_like(x, v) for x in f] for f, v in ((w.E, E), (w.T, T), (w.z, 1.0)))
    return w


@pytest.mark.parametrize("graph", [0, 1])
def test_nan_of_a_krylov_vector_is_not_a_solved_system(graph):
    """kappa beyond float's range: the single-precision cycle returns NaN
    while the residual of the uniform state is finite.  A NaN norm is neither
    below the tolerance nor an exact breakdown, so the cycle of 4 vectors is
    run to its end, and the step is refused."""
    w = _uniform((8, 8, 8), 1e39, T=0.9)
    H = make(w, precision=1, gmres_restart=4, use_graph=graph)
    rc, st = H.implicit_step([1e-3], raise_on_fail=False)
    assert rc != 0
    assert st[0]["krylov_iters"] == 4


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_norms_formed_from_the_vector_leave_other_problems_alone(precision, graph):
    """Beside a problem whose Krylov vectors are NaN and one whose first one
    lies in the span of the basis to rounding (a step so short that the
    operator is the identity): a third takes the iterations it takes alone."""
    bad, short, good = _uniform((8, 8, 8), 1e39, T=0.9), _box((10, 14, 6), 5), _box((16, 16, 16), 6)
    if not precision:                      # (finite in float64)
        bad = _box((8, 8, 8), 7)
    ws, dts = [bad, short, good], [1e-3, 1e-13, 1e-3]
    boxes = [I.Box(p, 0, (0, 0, 0), x.boxes[0].hi) for p, x in enumerate(ws)]
    w = I.Workload("three", [x.problems[0] for x in ws], boxes, [x.z[0] for x in ws],
                   [x.E[0] for x in ws], [x.T[0] for x in ws], np.array(dts))
    opt = dict(precision=precision, gmres_restart=4, use_graph=graph)
    rc, st = make(w, **opt).implicit_step(dts, raise_on_fail=False)
    alone = make(good, **opt).implicit_step([dts[2]])[1][0]
    assert (rc != 0) == bool(precision)
    assert st[2]["krylov_per_newton"] == alone["krylov_per_newton"]
    assert st[2]["newton_iters"] == alone["newton_iters"]
    assert set(st[1]["krylov_per_newton"]) <= {0, 1}


@pytest.mark.parametrize("kappa", [1e36, 4e36])
def test_sweeps_divide_by_diagonals_of_floats_whole_range(kappa):
    """Level sweeps (base level smoothed) whose diagonals lie between 2^126
    and float's largest value (3 to 6 faces of 3.2e37), and beyond it (each
    face 1.3e38): quotients to single precision of four operations, and 0."""
    w = _uniform((8, 8, 8), kappa)
    s = system(w, fac_base="smooth")
    H = make(w, precision=1, fac_base=1, gmres_restart=2)
    dt = 0.5                               # beta / h^2 = 32
    H.begin_step([dt])
    u = state(s, w)
    wv = np.concatenate([np.zeros(s.nc),
                         1e30 * np.random.default_rng(4).uniform(1.0, 2.0, s.nc)])
    H.precond_setup(native_from_compact(H, u))
    got = compact_from_native(H, H.precond_apply(native_from_compact(H, wv), H.native()))
    if kappa > 1e36:
        np.testing.assert_array_equal(got, 0.0)
        return
    ref = s.precond(u, dt)[0](wv)
    for f in (slice(0, s.nc), slice(s.nc, 2 * s.nc)):
        assert rel_err(got[f], ref[f]) < 1e-6


def test_tuned_shapes_are_kept_per_kernel(tmp_path):
    """One box shape alone (16 plane runs: staged planes) and 13 of it (208:
    wave runs) under one cache file: each kernel's choice is timed by itself
    and found again."""
    cache = str(tmp_path / "tiles.txt")
    few, many = _grid([(16, 16, 16)], []), _grid([(16, 16, 16)] * 13, [])
    assert [make(w).autotune(cache) for w in (few, many, few, many)] == [1, 1, 0, 0]


def test_large_hierarchies_are_tuned_in_few_launches():
    """Eight shapes of 96 and 128 cells (16 planes by default, so three other
    plane counts are tried): 12 launches for each of them and the lists of their
    tiles, together the time of 17.5; with the counts of small grids 20 and 27."""
    exts = [(96 + 32 * (s & 1), 96 + 16 * (s & 2), 96 + 8 * (s & 4)) for s in range(8)]
    w = _grid(exts, [])
    H = make(w)
    H.begin_step([1e-4] * 8)
    u, F = native_from_compact(H, np.concatenate([np.concatenate([x.ravel(order="F") for x in f])
                                                  for f in (w.E, w.T)])), H.native()
    t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    with torch.cuda.stream(H.stream):
        H.residual(u, F)
        t0.record()
        for _ in range(20):
            H.residual(u, F)
        t1.record()
    torch.cuda.synchronize()
    each = 1e-3 * t0.elapsed_time(t1) / 20
    tune = []
    for _ in range(3):
        start = time.perf_counter()
        assert H.autotune(None) == 8
        tune.append(time.perf_counter() - start)
    print(f"residual {1e6 * each:.0f} us, tuned in {1e3 * min(tune):.1f} ms")
    assert min(tune) < 8 * 22 * each


def test_steps_of_hundreds_of_problems():
    """300 problems at once, whose arrays do not fit one launch's arguments,
    against batches of 60, which do: the same systems to the same relative
    tolerances, so the states agree to the steps' own (1e-11 of the first
    residual; inner products are summed in other groups)."""
    exts = [(6, 6, 6), (8, 6, 6), (6, 8, 10)]
    ws = [_box(exts[p % 3], seed=200 + p) for p in range(300)]
    dts = [2e-4 * (1 + p % 7) for p in range(300)]

    def run(ps):
        w = I.Workload("many", [ws[p].problems[0] for p in ps],
                       [I.Box(i, 0, (0, 0, 0), exts[p % 3]) for i, p in enumerate(ps)],
                       [ws[p].z[0] for p in ps], [ws[p].E[0] for p in ps],
                       [ws[p].T[0] for p in ps], np.array([dts[p] for p in ps]))
        H = make(w, newton_rtol=1e-11, newton_atol=1e-18)
        its = [[st["newton_iters"] for st in H.implicit_step([dts[p] for p in ps])[1]]
               for _ in range(2)]
        E, T = H.get_fields()
        u = np.concatenate([E.cpu().numpy(), T.cpu().numpy()])
        return [u[i] for i in problem_slices(w)], its

    got, its = run(range(300))
    assert len(set(its[0])) > 1            # the mask of active problems changes
    for a in range(0, 300, 60):
        want, _ = run(range(a, a + 60))
        for p in range(60):
            assert rel_err(got[a + p], want[p]) < 1e-9


@pytest.mark.parametrize("precision", [0, 1])
def test_ghosts_of_large_tables(precision):
    """Twelve problems refined on half their domain by 4^3 boxes (2.2 M ghosts,
    siblings and coarse-fine: a thread takes both fields) against one of them
    alone (a field per block): residual, Jacobian action by one kernel, and
    preconditioner, bit for bit the same."""
    nprob, fine = 12, [(x, y, z) for z in range(0, 64, 4) for y in range(0, 64, 4)
                       for x in range(0, 32, 4)]
    one = _grid([(32, 32, 32)], [(f, tuple(c + 4 for c in f)) for f in fine])
    many = I.Workload("many", one.problems * nprob,
                      [I.Box(p, b.level, b.lo, b.hi) for p in range(nprob) for b in one.boxes],
                      one.z * nprob, one.E * nprob, one.T * nprob, np.full(nprob, 1e-3))
    rng = np.random.default_rng(5)
    n = one.ncells()
    v0 = rng.standard_normal(2 * n)
    u0 = np.concatenate([one.compact(one.E), one.compact(one.T)]) * rng.uniform(0.9, 1.1, 2 * n)

    def outputs(w, batch):
        H = make(w, precision=precision, stencil=0, gmres_restart=2)
        H.begin_step([1e-3] * len(w.problems))
        u = native_from_compact(H, batch(u0))
        v = batch(v0)
        out = [compact_from_native(H, H.residual(u, H.native())),
               compact_from_native(H, H.jvp(u, native_from_compact(H, v), H.native()))]
        H.precond_setup(u)
        return out + [compact_from_native(H, H.precond_apply(native_from_compact(H, v),
                                                             H.native()))]

    want = outputs(one, lambda x: x)
    got = outputs(many, lambda x: np.concatenate([np.tile(x[:n], nprob), np.tile(x[n:], nprob)]))
    for a, b in zip(got, want):
        for p in (0, nprob - 1):
            np.testing.assert_array_equal(a.reshape(2, nprob, n)[:, p].ravel(), b)


# 46 080 and 54 272 one-plane tiles: wave runs, staged planes
@pytest.mark.parametrize("width", [44, 52])
def test_stencil_kernel_of_large_refined_hierarchies(width):
    """The default kernel on both sides of its rule for several levels against
    one thread per cell, bounds as for the other sizes."""
    _one_kernel([(64, 64, 64)], [((x, y, z), (x + 4, y + 4, z + 4)) for z in range(0, 128, 4)
                                 for y in range(0, 128, 4) for x in range(0, width, 4)])


def _with_cycle(monkeypatch, m, n):
    """The oracle's multigrid as V(m, n)."""
    orig = pc.mg_vcycle
    monkeypatch.setattr(pc, "mg_vcycle", lambda grids, beta, rhs, level=0, nu_pre=1, nu_post=1,
                        cache=None: orig(grids, beta, rhs, level, m, n, cache))


# grids swept one by one, in blocks and within one workgroup (none, one and
# two of them), on colour-split storage and a base grid of two boxes
@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-4)])
@pytest.mark.parametrize("nu", [(2, 1), (1, 2), (1, 0), (2, 0), (3, 2)])
@pytest.mark.parametrize("grid", ["8", "12x12x12", "24x24x56", "64x32x32", "two boxes",
                                  "two levels"])
def test_precond_of_any_multigrid_cycle(monkeypatch, grid, nu, precision, tol):
    """Preconditioner with m sweeps before and n after each coarse correction
    against the oracle's V(m, n), tolerances as for V(1, 1)."""
    if grid == "two levels":
        w = I.static_amr(base=16, nlevels=2, side=(8, 16), state="front")
    elif grid == "two boxes":
        w = _grid([(24, 24, 24)], [])
        w.boxes = [I.Box(0, 0, (0, 0, 0), (10, 24, 24)), I.Box(0, 0, (10, 0, 0), (24, 24, 24))]
        w.E, w.T, w.z = ([x[0][:10], x[0][10:]] for x in (w.E, w.T, w.z))
    else:
        ext = tuple(int(x) for x in grid.split("x"))
        w = _box(ext * 3 if len(ext) == 1 else ext)
    _with_cycle(monkeypatch, *nu)
    s = system(w)
    H = make(w, precision=precision, gmres_restart=2, mg_nu_pre=nu[0], mg_nu_post=nu[1])
    H.begin_step([1e-3])
    rng = np.random.default_rng(42)
    u = s.sync(state(s, w) * rng.uniform(0.9, 1.1, 2 * s.nc))
    wv = rng.standard_normal(u.shape)
    H.precond_setup(native_from_compact(H, u))
    got = compact_from_native(H, H.precond_apply(native_from_compact(H, wv), H.native()))
    ref = s.precond(u, 1e-3)[0](wv)
    for f in (slice(0, s.nc), slice(s.nc, 2 * s.nc)):
        m = s.composite[f]
        assert rel_err(got[f][m], ref[f][m]) < tol


@pytest.mark.parametrize("nu", [(2, 1), (1, 2)])
def test_large_batches_of_any_multigrid_cycle(nu):
    """A hierarchy large enough for the fused base sweeps of V(1, 1), under
    another cycle, which they do not serve: each problem's preconditioner
    beside the others and alone, bit for bit the same."""
    ws, w = _sweep_batch()
    n = [x.ncells() for x in ws]
    us = [np.concatenate([x.compact(x.E), x.compact(x.T)]) for x in ws]
    vs = [np.random.default_rng(60 + p).standard_normal(2 * n[p]) for p in range(len(ws))]

    def apply(w, u, v):
        H = make(w, precision=1, gmres_restart=2, mg_nu_pre=nu[0], mg_nu_post=nu[1])
        H.begin_step([float(x) for x in w.dt])
        H.precond_setup(native_from_compact(H, u))
        return compact_from_native(H, H.precond_apply(native_from_compact(H, v), H.native()))

    got = apply(w, np.concatenate([x[:k] for x, k in zip(us, n)] + [x[k:] for x, k in zip(us, n)]),
                np.concatenate([x[:k] for x, k in zip(vs, n)] + [x[k:] for x, k in zip(vs, n)]))
    at = np.concatenate([[0], np.cumsum(n)])
    for p in range(1, len(ws)):
        want = apply(ws[p], us[p], vs[p])
        mine = np.concatenate([got[f + at[p]:f + at[p + 1]] for f in (0, at[-1])])
        np.testing.assert_array_equal(mine, want, err_msg=str(p))


# wave runs of 80^3 take two planes per tile (2000 plane runs), staged planes
# of 7 and 11 of them eight and sixteen (14 000 and 22 000)
@pytest.mark.parametrize("nprob,other", [(1, 4), (7, 4), (11, 8)])
def test_every_chunk_of_the_size_rule_keeps_every_value(nprob, other):
    """The default planes per tile give bit for bit another chunk's values."""
    w = _grid([(80, 80, 80)] * nprob, [])
    rng = np.random.default_rng(5)
    n = w.ncells()
    v = rng.standard_normal(2 * n)
    u = np.concatenate([w.compact(w.E), w.compact(w.T)]) * rng.uniform(0.9, 1.1, 2 * n)
    outs = []
    for zc in (0, other):
        H = make(w, stencil=3, zchunk=zc, gmres_restart=2)
        H.begin_step([float(x) for x in w.dt])
        F = H.residual(native_from_compact(H, u), H.native())
        Jv = H.jvp(native_from_compact(H, u), native_from_compact(H, v), H.native())
        outs.append((compact_from_native(H, F), compact_from_native(H, Jv)))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])


def test_precond_apply_needs_its_vectors():
    """The solver's own calls leave the input in place and pass none; a caller
    without one is refused rather than given the last call's."""
    from paper_1302_6303_amd import nrd
    H = make(_box((8, 8, 8)), gmres_restart=2)
    H.begin_step([1e-3])
    y = H.native()
    for w, out in ((None, y.data_ptr()), (y.data_ptr(), None)):
        assert nrd.nrd_precond_apply(H.h, w, out) == nrd.NRD_EINVAL


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("opt", [dict(), dict(fac_cycle=1), dict(fac_smoother=1),
                                 dict(fac_smoother=2), dict(fac_base=1)])
def test_workspaces_of_more_than_2_to_32_values(monkeypatch, opt, precision):
    """A workspace of 34.4 GB full of NaN and -1 (adjoint slots of a small
    refined hierarchy) is cleared as a small one is: ghost slots that nothing
    fills, and the counters of the sums.  Operators, preconditioner and a
    step, bit for bit those of a small clean workspace."""
    import torch
    w = I.static_amr(base=16, nlevels=3, side=(8, 16), state="front")
    plain = torch.empty
    rng = np.random.default_rng(5)
    n = w.ncells()
    v = rng.standard_normal(2 * n)
    u = np.concatenate([w.compact(w.E), w.compact(w.T)]) * rng.uniform(0.9, 1.1, 2 * n)

    def outputs(**more):
        H = make(w, precision=precision, **opt, **more)
        H.begin_step([1e-3])
        un = native_from_compact(H, u)
        out = [compact_from_native(H, H.residual(un, H.native())),
               compact_from_native(H, H.jvp(un, native_from_compact(H, v), H.native()))]
        H.precond_setup(un)
        out.append(compact_from_native(H, H.precond_apply(native_from_compact(H, v), H.native())))
        H.implicit_step([1e-4])
        out += [x.cpu().numpy() for x in H.get_fields()]
        return out, H.native_len, H.workspace_bytes

    want, nl, small = outputs()
    slots = -(-(8 * 2 ** 32 - small) // (16 * nl)) + 1
    monkeypatch.setattr(torch, "empty", lambda *a, **k: plain(*a, **k).fill_(255)
                        if k.get("dtype") == torch.uint8 else plain(*a, **k))
    got, _, large = outputs(adjoint_slots=slots)
    torch.cuda.empty_cache()
    assert large > 8 * 2 ** 32
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)

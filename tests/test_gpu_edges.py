"""Edges of the solver's ranges: overflow and NaN, cycles other than V(1,1),
hundreds of problems, the tile tuner's cache."""
import numpy as np
import pytest

from paper_1302_6303_amd import inputs as I
from tests.gpu_helpers import make
from tests.test_gpu_paths import _box

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

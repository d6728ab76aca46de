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


# plane runs of 256 cells times planes: 24, 1152 (one plane per tile),
# 3456 (two), 8192 (four)
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

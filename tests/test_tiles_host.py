"""Reduction tiles of the host tables (no device calls)."""
import pytest

from paper_1302_6303_amd import inputs as I


def test_dot_noalloc_takes_every_hierarchy_that_2048_cell_tiles_let_it():
    """Finer reduction tiles give small grids more workgroups, but a hierarchy
    of thousands of boxes must not outgrow nrd_dot_noalloc's fixed array of
    32768 tiles by them: 100 boxes of 1728 cells and 32600 of one.  (Without a
    workspace an accepted call ends at its state check.)"""
    from paper_1302_6303_amd import nrd
    exts = [(12, 12, 12)] * 100 + [(1, 1, 1)] * 32600
    H = nrd.Hierarchy([I.Problem(e) for e in exts],
                      [I.Box(p, 0, (0, 0, 0), e) for p, e in enumerate(exts)],
                      nrd.default_options(), bind=False)
    assert nrd.nrd_dot_noalloc(H.h, None, None, None) == nrd.NRD_ESTATE


@pytest.mark.parametrize("hi", [(2 ** 31 - 1, 4, 4), (-2 ** 31, 4, 4), (2 ** 31 - 1,) * 3])
def test_boxes_of_absurd_extents_are_refused(hi):
    from paper_1302_6303_amd import nrd
    with pytest.raises(nrd.NrdError):
        nrd.Hierarchy([I.Problem((4, 4, 4))], [I.Box(0, 0, (-2 ** 31, 0, 0), hi)],
                      nrd.default_options(), bind=False)

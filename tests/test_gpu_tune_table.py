"""The autotune table is read by every grid of a size class: it holds shapes
that are candidates for all of them, or says that each takes its default."""
import json

import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu

LISTED = {"2d": {2, 3, 4, 5, 6, 8, 12, 16, 32, 64}, "2d_ns": {2, 3, 4, 5, 6, 8, 12, 16, 32, 64},
          "3d": {8, 12, 16, 20, 24, 28, 32, 40, 48, 52, 56, 64}, "3d_gen": {4, 8, 12, 16, 24, 32, 48, 64}}


def viscous(*a):
    case = CS.inlet_case(*a)
    case.params = CS.Params(**{**case.params.__dict__, "mu": 1e-2})
    return case


def box(ni, nj, nk):
    case = CS.blobs_case(max(ni, nj, nk), nblobs=3)
    b = case.blocks[0]
    case.U0 = [np.ascontiguousarray(case.U0[0][:, :nk, :nj, :ni])]
    b.ni, b.nj, b.nk = ni, nj, nk
    return case


# kernel, a grid, another of its size class (and kernel)
PAIRS = {
    "2d": (lambda: CS.vortex_2d(70, 60), lambda: CS.vortex_2d(64, 90)),
    "2d_ns": (lambda: viscous(128, 45, 1), lambda: viscous(72, 100, 1)),
    "3d": (lambda: box(20, 20, 20), lambda: box(18, 16, 26)),
    "3d_gen": (lambda: CS.curv3d_case(20, 18, 14, nblocks=1), lambda: CS.curv3d_case(12, 20, 30, nblocks=1)),
}


def key_of(kind, case):
    return f"{kind[:2]}_fp64_c{case.ncells.bit_length() - 1}{kind[2:]}"


def shape_of(g, case):
    g.set_state(case.state_flat())
    g.residual(case.params)
    st = g.stats()
    return st["tile_rows"], st["tile_ny"], st["tiles"]


@pytest.mark.parametrize("kind", sorted(PAIRS))
def test_zero_rows_are_each_grids_default(kind, tmp_path, monkeypatch):
    from paper_2305_18057_amd import fv
    path = tmp_path / "t.json"
    for make in PAIRS[kind]:
        case = make()
        monkeypatch.delenv("FV_AUTOTUNE_CACHE", raising=False)
        default = shape_of(fv.Grid(case), case)
        path.write_text(json.dumps({key_of(kind, case): {"rows": 0, "ny": 0, "ms": 1.0}}))
        monkeypatch.setenv("FV_AUTOTUNE_CACHE", str(path))
        g = fv.Grid(case)
        assert shape_of(g, case) == default
        g.tune(case.params)
        assert shape_of(g, case) == default


@pytest.mark.parametrize("kind", sorted(PAIRS))
def test_a_tuned_table_fits_the_class(kind, tmp_path, monkeypatch):
    """What the tuner records for one grid is a listed candidate or "default",
    never a number fitted to that grid; a later handle gets the tuned shape."""
    from paper_2305_18057_amd import fv
    monkeypatch.delenv("FV_AUTOTUNE_CACHE", raising=False)
    case, other = PAIRS[kind][0](), PAIRS[kind][1]()
    key = key_of(kind, case)
    assert key == key_of(kind, other)
    path = tmp_path / "t.json"
    g = fv.Grid(case)
    g.set_state(case.state_flat())
    tuned = g.tune(case.params, str(path))
    entry = json.loads(path.read_text())[key]
    assert entry["rows"] in LISTED[kind] | {0}
    default = shape_of(fv.Grid(other), other)
    monkeypatch.setenv("FV_AUTOTUNE_CACHE", str(path))
    assert shape_of(fv.Grid(case), case) == (tuned["tile_rows"], tuned["tile_ny"], tuned["tiles"])
    if entry["rows"] == 0:
        assert shape_of(fv.Grid(other), other) == default

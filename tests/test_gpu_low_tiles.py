"""Tiles of one row or one plane, which small grids get by default: bitwise the
state of tall tiles, in every kernel and on the allocation-free path; and a
grid that is stepped with and without a viscosity keeps a list for each."""
import json

import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


def with_rows(monkeypatch, tmp_path, case, rows, ny=1):
    from paper_2305_18057_amd import fv
    key = f"{case.ndim}d_fp64_c{case.ncells.bit_length() - 1}" + ("_gen" if case.name.startswith("curv") else "")
    path = tmp_path / f"{key}_{rows}_{ny}.json"
    path.write_text(json.dumps({key: {"rows": rows, "ny": ny, "ms": 0.0}}))
    monkeypatch.setenv("FV_AUTOTUNE_CACHE", str(path))
    g = fv.Grid(case)
    monkeypatch.delenv("FV_AUTOTUNE_CACHE")
    assert g.stats()["tile_rows"] == rows
    return g


def stepped(g, case, prm, n=3):
    g.set_state(case.state_flat())
    g.step(prm, n)
    return g.get_state()


@pytest.mark.parametrize("limiter,rk", [(CS.MINMOD, 3), (CS.UNLIMITED, 4)])
@pytest.mark.parametrize("make", [
    lambda: CS.inlet_case(136, 19, 2), lambda: CS.vortex_2d(70, 33),
    lambda: CS.blobs_case(20, nblobs=3), lambda: CS.curv3d_case(20, 9, 7, walls_k=True)])
def test_low_tiles_are_bitwise_the_tall_ones(monkeypatch, tmp_path, make, limiter, rk):
    from paper_2305_18057_amd import fv
    case = make()
    prm = CS.Params(**{**case.params.__dict__, "limiter": limiter, "rk": rk})
    shapes = [(1, 7), (1, 3), (2, 7), (64, 7)] if case.ndim == 3 else [(1, 1), (2, 1), (64, 1)]
    out = [stepped(with_rows(monkeypatch, tmp_path, case, *s), case, prm) for s in shapes]
    out.append(stepped(fv.Grid(case), case, prm))
    if case.ndim == 2:
        import torch
        U = torch.tensor(case.state_flat(), device="cuda")
        fv.step_noalloc(case, U, params=prm, nsteps=3)
        out.append(U.cpu().numpy())
    assert all(np.array_equal(out[0], o) for o in out[1:])


def test_a_viscosity_between_euler_calls():
    """Slip walls only: the Euler kernel's tiles without a viscosity, the
    Navier-Stokes kernel's with one, in turn on one handle."""
    from paper_2305_18057_amd import fv
    case = CS.inlet_case(128, 24, 1)
    eu, ns = case.params, CS.Params(**{**case.params.__dict__, "mu": 1e-2})
    ref = {}
    for name, p in (("eu", eu), ("ns", ns)):
        ref[name] = stepped(fv.Grid(case), case, p)
    g = fv.Grid(case)
    rows = set()
    for name, p in (("eu", eu), ("ns", ns), ("eu", eu), ("ns", ns)):
        assert np.array_equal(stepped(g, case, p), ref[name])
        rows.add((name, g.stats()["tile_rows"]))
    assert len(rows) == 2 and len({r for _, r in rows}) == 2

"""Each tile list of a 2D grid takes the tuned shape of its own kernel: a table
that holds the Euler kernel's shape alone leaves the Navier-Stokes list at its
default, and the other way round."""
import json

import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu

EULER, NS = 3, 5  # rows in the tables; neither is a default of these grids


def noslip_case():
    case = CS.inlet_case(128, 48, 1)
    for b in case.blocks:
        b.bc[2] = b.bc[3] = CS.BC(CS.NOSLIP)
    return case


def source_case():
    case = CS.inlet_case(128, 48, 1)
    case.source = [np.zeros_like(u) for u in case.U0]
    return case


def rows_of(case, p):
    """Tile rows of a handle made now, after a residual with parameters p."""
    from paper_2305_18057_amd import fv
    g = fv.Grid(case)
    g.set_state(case.state_flat())
    g.residual(p)
    return g.stats()["tile_rows"]


@pytest.mark.parametrize("which", ["euler", "ns", "both"])
@pytest.mark.parametrize("make", [lambda: CS.inlet_case(128, 48, 1), noslip_case, source_case])
def test_each_list_takes_its_own_shape(make, which, tmp_path, monkeypatch):
    case = make()
    eu = case.params
    visc = CS.Params(**{**eu.__dict__, "mu": 1e-2})
    monkeypatch.delenv("FV_AUTOTUNE_CACHE", raising=False)
    default = {n: rows_of(case, p) for n, p in (("eu", eu), ("ns", visc))}
    assert not {EULER, NS} & set(default.values())
    key = f"2d_fp64_c{case.ncells.bit_length() - 1}"
    table = {}
    if which != "ns":
        table[key] = {"rows": EULER, "ny": 1, "ms": 0.0}
    if which != "euler":
        table[key + "_ns"] = {"rows": NS, "ny": 1, "ms": 0.0}
    path = tmp_path / "t.json"
    path.write_text(json.dumps(table))
    monkeypatch.setenv("FV_AUTOTUNE_CACHE", str(path))
    ns = default["ns"] if which == "euler" else NS
    # a wall or a source: every call runs the Navier-Stokes kernel
    plain = make in (noslip_case, source_case)
    assert rows_of(case, visc) == ns
    assert rows_of(case, eu) == (ns if plain else default["eu"] if which == "ns" else EULER)

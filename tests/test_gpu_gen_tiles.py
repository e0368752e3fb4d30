"""The general 3D kernel's tiles: blocks whose sides leave ragged tiles, tiles
one cell wide or high, more planes than one tile, and small ones; walls and
links.  Against the oracle, and bitwise the same for every tile height."""
import json

import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ni,nj,nk,nblocks,walls", [
    (2, 2, 2, 1, False), (61, 3, 5, 1, True), (130, 2, 4, 1, False), (16, 15, 9, 1, True),
    (48, 33, 4, 2, False), (24, 70, 3, 3, True), (8, 2, 70, 1, False), (16, 16, 67, 2, True)])
def test_gen_tiles(tmp_path, monkeypatch, ni, nj, nk, nblocks, walls):
    from oracle import oracle as O
    from paper_2305_18057_amd import fv
    case = CS.curv3d_case(ni, nj, nk, nblocks=nblocks, walls_k=walls)
    ref = O.OracleGrid(case)
    Ro, _, scale = ref.residual(case.params, with_scale=True)
    ref.run(case.params, 2)
    Uo, states = ref.get_state(), []
    cls = case.ncells.bit_length() - 1
    for rows in (4, 16, 64):
        path = tmp_path / f"t{rows}.json"
        path.write_text(json.dumps({f"3d_fp64_c{cls}_gen": {"rows": rows, "ny": 4, "ms": 0.0}}))
        monkeypatch.setenv("FV_AUTOTUNE_CACHE", str(path))
        g = fv.Grid(case)
        st = g.stats()
        w, h = st["tile_cols"], st["tile_ny"]
        assert st["tile_rows"] == rows
        assert max((w + 1) * h, w * (h + 1), 4 * (w + h)) <= 256
        g.set_state(case.state_flat())
        Rg, _ = g.residual(case.params)
        assert P.residual_err(case, Rg, Ro, scale) <= P.FP64_TOL
        g.step(case.params, 2)
        states.append(g.get_state())
        assert P.state_err(case, states[-1], Uo) <= P.FP64_TOL
    assert np.array_equal(states[0], states[1]) and np.array_equal(states[0], states[2])

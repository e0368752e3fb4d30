"""The allocation-free step at the limit of its scratch: every grid whose
layout with the lowest reserved tiles fits is stepped, also where its tile list
is longer than that."""
import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


def boxes(n, ni, nj, nk):
    """n separate small boxes of ni x nj x nk cells, with node coordinates."""
    k, j, i = np.meshgrid(*(np.arange(m + 1.0) for m in (nk, nj, ni)), indexing="ij")
    prim = (1.0, 0.6, 0.3, 0.0, 1.0 / CS.GAMMA)
    rng = np.random.default_rng(7)
    ext = [CS.BC(CS.EXTRAP)] * 6
    blocks, U0 = [], []
    for _ in range(n):
        blocks.append(CS.Block(ni, nj, nk, i, j, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), ext, k))
        U = CS.conserved(1.0 + 0.01 * rng.standard_normal((nk, nj, ni)), prim[1:4], prim[4])
        U0.append(np.stack([np.broadcast_to(u, (nk, nj, ni)) for u in U]))
    return CS.Case("boxes", 3, blocks, U0, CS.Params(qref=CS.qref_of(prim, 3)), 1)


@pytest.mark.parametrize("ni,nj,nk", [(64, 2, 2), (61, 1, 4), (64, 3, 4)])
def test_the_largest_grid_that_fits_is_stepped(ni, nj, nk):
    import torch
    from paper_2305_18057_amd import fv

    def step(n):
        case = boxes(n, ni, nj, nk)
        U = torch.tensor(case.state_flat(), device="cuda")
        return case, U, fv.step_noalloc(case, U, nsteps=1, check=False)["status"]

    lo, hi = 1, 2 * (64 << 20) // (80 * ni * nj * nk)  # fits, does not
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if step(mid)[2] == fv.FV_E_NOMEM else (mid, hi)
    for n in (lo, lo - 1, lo - 7):
        case, U, status = step(n)
        assert status == fv.FV_OK, (n, status)
    g = fv.Grid(case)
    g.set_state(case.state_flat())
    g.step(case.params, 1)
    assert np.array_equal(U.cpu().numpy(), g.get_state())

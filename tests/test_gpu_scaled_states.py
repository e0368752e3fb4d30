"""The Euler flux is homogeneous of degree one in the conserved state: a state
scaled by a power of four (so that roots of the density scale exactly too) has
the residual scaled by it, bit for bit, as far as the type's range reaches."""
import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limiter", [CS.MINMOD, CS.UNLIMITED])
@pytest.mark.parametrize("make", [lambda: CS.vortex_2d(70, 9), lambda: CS.inlet_case(72, 10, 1),
                                  lambda: CS.blobs_case(12, nblobs=2), lambda: CS.curv3d_case(12, 8, 8)])
def test_residual_of_a_scaled_state(make, limiter):
    from paper_2305_18057_amd import fv
    case = make()
    rng = np.random.default_rng(8)
    case.U0 = [u * (1.0 + 0.01 * rng.standard_normal(u.shape)) for u in case.U0]
    for b in case.blocks:  # (an inflow state would have to be scaled too)
        b.bc = [CS.BC(CS.EXTRAP) if c.kind == CS.INFLOW else c for c in b.bc]
    prm = CS.Params(**{**case.params.__dict__, "limiter": limiter})
    g = fv.Grid(case)
    U = case.state_flat()
    g.set_state(U)
    R = g.residual(prm)[0]
    dt = g.step(prm, 1)["dt_last"]
    V = g.get_state()
    for s in (2.0 ** 520, 2.0 ** -520, 2.0 ** 20):
        g.set_state(s * U)
        assert np.array_equal(g.residual(prm)[0], s * R), s
        assert g.step(prm, 1)["dt_last"] == dt, s
        assert np.array_equal(g.get_state(), s * V), s

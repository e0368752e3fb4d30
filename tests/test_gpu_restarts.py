"""A run that is interrupted goes on bitwise as the run that is not: the limit
of the time step formed by the last stage and the one formed for a state that
is set (or kept through tuning) are the same number, in every stage kernel."""
import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu

CASES = {
    "inlet": lambda: CS.inlet_case(96, 24, 2),
    "vortex": lambda: CS.vortex_2d(48, 32),
    "viscous": lambda: with_params(CS.inlet_case(96, 24, 2), mu=1e-2),
    "blobs": lambda: CS.blobs_case(16, nblobs=3),
    "curved": lambda: CS.curv3d_case(16, 10, 8),
    "curved_source": lambda: CS.curv3d_case(12, 10, 8, state="mms"),
}


def with_params(case, **kw):
    case.params = CS.Params(**{**case.params.__dict__, **kw})
    return case


def noisy(name, seed):
    """The case with 2% seeded noise on every variable, so that another cell
    sets the time step for every seed."""
    case = CASES[name]()
    rng = np.random.default_rng(seed)
    case.U0 = [np.ascontiguousarray(u * (1.0 + 0.02 * rng.standard_normal(u.shape))) for u in case.U0]
    return case


@pytest.mark.parametrize("precision", [CS.FP64, CS.FP32_FLUX])
@pytest.mark.parametrize("name", sorted(CASES))
def test_restart_is_bitwise(name, precision):
    """Six noisy states, eight restarts each: after every step the state goes
    into a second handle, which takes the next step from it."""
    from paper_2305_18057_amd import fv
    for seed in range(6):
        case = with_params(noisy(name, seed), precision=precision)
        a, b = fv.Grid(case), fv.Grid(case)
        a.set_state(case.state_flat())
        a.step(case.params, 1)
        for n in range(8):
            b.set_state(a.get_state())
            ia, ib = a.step(case.params, 1), b.step(case.params, 1)
            assert ia["dt_last"] == ib["dt_last"], (seed, n)
            assert np.array_equal(a.get_state(), b.get_state()), (seed, n)


@pytest.mark.parametrize("name", ["inlet", "viscous", "blobs", "curved"])
def test_tuning_between_steps_keeps_the_run(name, tmp_path):
    from paper_2305_18057_amd import fv
    for seed in range(3):
        case = noisy(name, seed)
        a, b = fv.Grid(case), fv.Grid(case)
        for n, g in enumerate((a, b)):
            g.set_state(case.state_flat())
            g.step(case.params, 3)
            if n:
                g.tune(case.params, str(tmp_path / f"{seed}.json"))
            g.step(case.params, 3)
        assert np.array_equal(a.get_state(), b.get_state()), seed


def test_switching_precision_between_steps_keeps_the_run():
    """An FP32-flux step after FP64 steps takes the time step that the state
    itself gives."""
    from paper_2305_18057_amd import fv
    for seed in range(6):
        case = noisy("inlet", seed)
        p32 = CS.Params(**{**case.params.__dict__, "precision": CS.FP32_FLUX})
        a, b = fv.Grid(case), fv.Grid(case)
        a.set_state(case.state_flat())
        a.step(case.params, 2)
        b.set_state(a.get_state())
        assert a.step(p32, 1)["dt_last"] == b.step(p32, 1)["dt_last"]
        assert np.array_equal(a.get_state(), b.get_state())

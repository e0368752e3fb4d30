"""The viscous flux through a link of two blocks is the flux the uncut grid has
there, bit for bit, so both blocks take the same one."""
import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


def field(Ni, Nj, seed):
    prim = (1.0, 0.5, 0.1, 0.0, 1.0 / CS.GAMMA)
    rng = np.random.default_rng(seed)

    def f(mean):
        return mean + 0.02 * rng.standard_normal((Nj, Ni))
    return prim, CS.conserved(f(1.0), [f(0.5), f(0.1)], f(prim[4]))[:, None]


def cut_case(cuts_i, cuts_j, walls, origin, seed=2):
    """A wavy mesh in blocks [cuts_i] x [cuts_j] (their sizes), inflow to
    outflow in i, walls in j; the mesh's corner at `origin`."""
    Ni, Nj = sum(cuts_i), sum(cuts_j)
    X, Y = CS.inlet_mesh(Ni, Nj, Lx=0.02 * Ni, Ly=0.02 * Nj, wave=0.007, shear=0.3)
    X, Y = X + origin[0], Y + origin[1]
    prim, U = field(Ni, Nj, seed)
    wall = CS.BC(walls, prim=(0.0, 0.1, 0.0, 0.0, 0.0))
    ni, nj = len(cuts_i), len(cuts_j)
    oi, oj = np.cumsum([0] + cuts_i), np.cumsum([0] + cuts_j)
    blocks, U0 = [], []
    for bj in range(nj):
        for bi in range(ni):
            me = bj * ni + bi
            bc = [CS.BC(CS.BLOCK, me - 1, CS.IMAX) if bi else CS.BC(CS.INFLOW, prim=prim),
                  CS.BC(CS.BLOCK, me + 1, CS.IMIN) if bi < ni - 1 else CS.BC(CS.EXTRAP),
                  CS.BC(CS.BLOCK, me - ni, 3) if bj else wall,
                  CS.BC(CS.BLOCK, me + ni, 2) if bj < nj - 1 else wall,
                  CS.BC(CS.PERIODIC), CS.BC(CS.PERIODIC)]
            s = (slice(oj[bj], oj[bj + 1] + 1), slice(oi[bi], oi[bi + 1] + 1))
            c = (slice(None), slice(None), slice(oj[bj], oj[bj + 1]), slice(oi[bi], oi[bi + 1]))
            blocks.append(CS.Block(cuts_i[bi], cuts_j[bj], 1, X[s].copy(), Y[s].copy(), (0.0, 0.0, 0.0),
                                   (1.0, 1.0, 1.0), bc))
            U0.append(np.ascontiguousarray(U[c]))
    prm = CS.Params(qref=CS.qref_of(prim, 2), mu=2e-3)
    return CS.Case("ns_cut", 2, blocks, U0, prm, 2)


def whole(case, flat, cuts_i, cuts_j):
    """The blocks' values as one array (var, j, i)."""
    parts = case.split_flat(np.asarray(flat))
    n = len(cuts_i)
    rows = [np.concatenate([p[:, 0] for p in parts[r * n:(r + 1) * n]], axis=2) for r in range(len(cuts_j))]
    return np.concatenate(rows, axis=1)


@pytest.mark.parametrize("precision", [CS.FP64, CS.FP32_FLUX])
@pytest.mark.parametrize("walls", [CS.NOSLIP, CS.SLIPWALL])
@pytest.mark.parametrize("cuts_i,cuts_j", [([64, 70], [33]), ([90], [17, 30]), ([2, 31, 64, 5], [2, 19, 3])])
@pytest.mark.parametrize("origin", [(0.0, 0.0), (37.0, -11.0)])
def test_a_cut_grid_has_the_uncut_grids_state(cuts_i, cuts_j, walls, precision, origin):
    from paper_2305_18057_amd import fv
    out = []
    for ci, cj in ((cuts_i, cuts_j), ([sum(cuts_i)], [sum(cuts_j)])):
        case = cut_case(ci, cj, walls, origin)
        p = CS.Params(**{**case.params.__dict__, "precision": precision, "dt_fixed": 2e-3})
        g = fv.Grid(case)
        g.set_state(case.state_flat())
        R, _ = g.residual(p)
        g.step(p, 5)
        out.append((whole(case, R, ci, cj), whole(case, g.get_state(), ci, cj)))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])

"""The stage launch holds every tile of a grid that fits the device at once."""
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case,per_wg", [
    (lambda: CS.vortex_2d(65, 9), 4), (lambda: CS.vortex_2d(200, 61), 4), (lambda: CS.vortex_2d(3, 2), 4),
    (lambda: CS.blobs_case(20, nblobs=1), 1), (lambda: CS.blobs_case(76, nblobs=1), 1),
    (lambda: CS.curv3d_case(42, 20, 35), 1)])
def test_no_tile_waits_for_a_second_round(case, per_wg):
    """Tiles that are no multiple of the eight parts of the list: the launch is
    rounded up to hold them, and stays a multiple of eight."""
    from paper_2305_18057_amd import fv
    c = case()
    g = fv.Grid(c)
    st = g.stats()
    chunk = -(-st["tiles"] // 8)  # the largest part
    assert st["launch_blocks"] % 8 == 0
    assert st["launch_blocks"] // 8 * per_wg >= chunk
    g.set_state(c.state_flat())
    assert g.step(c.params, 1)["steps"] == 1

"""A served uniform 3D box takes tiles of one greatest height, whether its shape
comes from a table (which holds shapes timed on a grid alone) or is the
default: seen in dry-run mode by the arena a request takes."""
import pytest

from paper_2305_18057_amd import cases as CS
from tests.test_server_low_tiles import arena_peak

KEY = "3d_fp32flux_c15"
LIMIT = 20  # planes


@pytest.mark.parametrize("ny", [3, 7])
def test_a_served_box_takes_no_taller_tiles(ny, tmp_path):
    from paper_2305_18057_amd import fv as fvb
    # 64 planes: 20 of them to a tile make 4 layers, 32 to 59 make 2
    case = CS.blobs_case(32)
    case.blocks[0].nk, case.blocks[0].ni = 64, 16
    case.U0 = [case.U0[0].reshape(5, 64, 32, 16)]
    at = {r: arena_peak(fvb, case, KEY, r, ny, tmp_path) for r in (8, LIMIT, 36, 59, 64)}
    assert at[36] == at[59] == at[64] == at[LIMIT] < at[8]
    if ny == 7:  # the j-rows of an untuned box
        assert arena_peak(fvb, case, "no such key", 8, ny, tmp_path) == at[LIMIT]

"""A request is refused for its size only when it does not fit with the tallest
tiles either: the smallest arena that takes it does not depend on the tile
shape it would get with more room.  Dry run."""
import json

import pytest

from paper_2305_18057_amd import cases as CS


def with_mu(case):
    case.params = CS.Params(**{**case.params.__dict__, "mu": 1e-2})
    return case


def smallest_arena(fvb, case, table):
    def takes(nbytes):
        try:
            srv = fvb.Server(arena_bytes=nbytes, max_instances=1, autotune_cache=table, dry_run=True)
        except fvb.FVError:
            return False
        try:
            srv.submit(case, drop_tol=0.0, max_steps=1)
        except fvb.FVError as e:
            assert e.status == fvb.FV_E_NOMEM
            return False
        finally:
            srv.close()
        return True

    lo, hi = 0, 64 << 20
    while hi - lo > 256:
        mid = (lo + hi) // 2 // 256 * 256
        lo, hi = (lo, mid) if takes(mid) else (mid, hi)
    return hi


@pytest.mark.parametrize("make, key, ny", [
    (lambda: with_mu(CS.inlet_case(64, 512, 1)), "2d_fp32flux_c15_ns", 1),
    (lambda: CS.inlet_case(128, 256, 1), "2d_fp32flux_c15", 1),
    (lambda: CS.blobs_case(32), "3d_fp32flux_c15", 7),
    (lambda: CS.curv3d_case(64, 22, 23, nblocks=1), "3d_fp32flux_c14_gen", 4)])
def test_the_smallest_arena_is_that_of_the_tallest_tiles(make, key, ny, tmp_path):
    from paper_2305_18057_amd import fv as fvb
    case = make()
    assert case.ncells.bit_length() - 1 == int(key.split("_c")[1].split("_")[0])
    table = tmp_path / "tall.json"
    table.write_text(json.dumps({key: {"rows": 64, "ny": ny, "ms": 1.0}}))
    assert smallest_arena(fvb, case, None) == smallest_arena(fvb, case, str(table))

"""A shape tuned for a grid of its own (down to single rows or planes) gives a
served instance tiles of 2 rows (2D), 8 planes (3D) or 4 (general 3D) at least:
seen in dry-run mode by the arena a request takes, which grows with its tiles."""
import json
import time

import pytest

from paper_2305_18057_amd import cases as CS


def arena_peak(fvb, case, key, rows, ny, tmp_path):
    table = tmp_path / f"{key}_{rows}.json"
    table.write_text(json.dumps({key: {"rows": rows, "ny": ny, "ms": 1.0}}))
    srv = fvb.Server(arena_bytes=64 << 20, max_instances=1, autotune_cache=str(table), dry_run=True)
    t = srv.submit(case, drop_tol=0.0, max_steps=2)
    t0 = time.time()
    while srv.poll(t) is None and time.time() - t0 < 20.0:
        time.sleep(0.001)
    peak = srv.stats()["arena_peak"]
    srv.close()
    return peak


@pytest.mark.parametrize("make, key, low, ny", [
    (lambda: CS.inlet_case(128, 96, 1), "2d_fp32flux_c13", 2, 1),
    (lambda: CS.blobs_case(32), "3d_fp32flux_c15", 8, 7),
    (lambda: CS.curv3d_case(40, 20, 32, nblocks=1), "3d_fp32flux_c14_gen", 4, 4),
])
def test_a_served_instance_takes_no_lower_tiles(make, key, low, ny, tmp_path):
    from paper_2305_18057_amd import fv as fvb
    case = make()
    at = {r: arena_peak(fvb, case, key, r, ny, tmp_path) for r in (1, low, 4 * low)}
    assert at[1] == at[low]
    assert at[4 * low] < at[low]  # (the table is read)

"""Making a handle of a grid of very many blocks: the general 3D kernel's tile
shapes cost no more than the rest of it."""
import ctypes as C
import time

import numpy as np
import pytest

from paper_2305_18057_amd import cases as CS

pytestmark = pytest.mark.gpu


def boxes(n, orient):
    """n uniform cubes in a row of links; orient turns every link (the general
    kernel) or none (the uniform one)."""
    blocks = []
    for b in range(n):
        bc = [CS.BC(CS.EXTRAP)] * 6
        if b:
            bc[0] = CS.BC(CS.BLOCK, b - 1, CS.IMAX, orient=orient)
        if b < n - 1:
            bc[1] = CS.BC(CS.BLOCK, b + 1, CS.IMIN, orient=orient)
        blocks.append(CS.Block(8, 8, 8, None, None, (8.0 * b, 0.0, 0.0), (1.0, 1.0, 1.0), bc))
    U0 = [np.zeros((5, 8, 8, 8))] * n
    return CS.Case("boxes", 3, blocks, U0, CS.Params(), 1)


def seconds(case):
    import torch
    from paper_2305_18057_amd import fv
    gd = fv.GridDesc(case)
    L = fv.lib()
    nbytes = L.fv_grid_workspace_bytes(C.byref(gd.desc), 0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    best = 1e9
    for _ in range(7):
        h = C.c_void_p()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        st = L.fv_create_grid(C.byref(gd.desc), C.c_void_p(ws.data_ptr()), C.c_size_t(nbytes), C.c_void_p(0),
                              C.byref(h))
        best = min(best, time.perf_counter() - t0)
        assert st == fv.FV_OK
        L.fv_destroy_grid(h)
    return best


def test_general_tiles_of_many_blocks_cost_no_more_than_the_rest():
    uniform, general = seconds(boxes(2000, 0)), seconds(boxes(2000, 2))
    print(f"  2000 blocks: {uniform * 1e6:.0f} us uniform, {general * 1e6:.0f} us general", flush=True)
    assert general < 2.0 * uniform

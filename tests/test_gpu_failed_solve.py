"""A solve that fails after it has queued work returns with that work done:
its workspace belongs to the caller again."""
import ctypes
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_nothing_writes_to_the_workspace_of_a_failed_solve():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    # the start points of every graph are drawn, a launch each and slower than
    # they are queued, before the tuner finds that no tile of 64 holds a graph
    G, n, B = 400, 2000, 512
    g = types.SimpleNamespace(n=G * n, row_ptr=np.zeros(G * n + 1, np.int32), col_idx=np.zeros(0, np.int32),
                              weight=None, vtx_offset=np.arange(G + 1, dtype=np.int64) * n)
    dg = mqo.DeviceGraph(g, DEV)
    p = mqo.make_params(batch=B, steps_per_round=1, rounds=1, plan="persistent", tile_cols=64, tile_vec=1)
    nbytes = mqo.lib().mqo_workspace_size(dg.struct, ctypes.byref(p), 0)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
    bx = torch.empty(G * n, dtype=torch.int8, device=DEV)
    bv = torch.empty(G, dtype=torch.int64, device=DEV)
    r = mqo._Result(bx.data_ptr(), bv.data_ptr(), None, None)
    for _ in range(3):
        ws.zero_()
        torch.cuda.synchronize()
        assert mqo.lib().mqo_solve_mis(dg.struct, ctypes.byref(p), None, ctypes.byref(r),
                                       ctypes.c_void_p(ws.data_ptr()), nbytes, mqo._stream(dg.device)) == -5
        ws.zero_()  # on the caller's stream, at once
        torch.cuda.synchronize()
        assert int(torch.count_nonzero(ws)) == 0

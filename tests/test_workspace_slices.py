"""The room for the persistent plan's slices in the workspace: part of the
size where a solve may use them, and of no other call."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from synth import graphs  # noqa: E402


@pytest.fixture(scope="module")
def mqo():
    from paper_2605_06921_amd import mqo as m
    return m


def size(mqo, n, nnz, kind=0, weight=None, **kw):
    off = np.array([0, n], dtype=np.int64)
    s = mqo._Graph()
    s.num_graphs, s.n_total, s.nnz_total = 1, n, nnz
    s.vtx_offset = off.ctypes.data_as(ctypes.POINTER(ctypes.c_int64))
    s.row_ptr, s.col_idx, s.weight = 0x1000, 0x1000, weight
    p = mqo.make_params(batch=4, **kw)
    p.maxcut_objective = kind
    return mqo.lib().mqo_workspace_size(ctypes.byref(s), ctypes.byref(p), kind)


def test_slices_are_part_of_the_size_where_they_may_run(mqo):
    n, nnz = 4000, 40000
    base = size(mqo, n, nnz, plan="batched")
    assert size(mqo, n, nnz, plan="plain") == base
    for plan in ("auto", "persistent"):
        assert size(mqo, n, nnz, plan=plan) > base + 288 * n
        assert size(mqo, n, nnz, kind=1, plan=plan) > base + 288 * n
        for fixed in (dict(tile_vec=1), dict(tile_csr=1), dict(tile_reg=1), dict(tile_sb=1)):
            assert size(mqo, n, nnz, plan=plan, **fixed) == base
        assert size(mqo, n, nnz, kind=1, weight=0x1000, plan=plan) == size(mqo, n, nnz, kind=1, weight=0x1000,
                                                                           plan="batched")
        for form in (2, 3, 4):  # formulations that the persistent plan does not run
            assert size(mqo, n, nnz, kind=form, plan=plan) == base
    assert size(mqo, 8193, nnz, plan="auto") == size(mqo, 8193, nnz, plan="batched")


@pytest.mark.gpu
@pytest.mark.parametrize("plan", ["persistent", "auto"])
def test_solve_without_room_for_slices(mqo, plan):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = graphs.concat([graphs.erdos_renyi(300, 0.1, 1), graphs.erdos_renyi(120, 0.2, 2)])
    dg = mqo.DeviceGraph(g, "cuda:0")
    kw = dict(batch=6, steps_per_round=100, rounds=2, alpha=0.02, rho=0.1, seed=4)
    mqo.lib().mqo_clear_caches()
    ref = mqo.solve("mis", dg, plan=plan, **kw)
    p = mqo.make_params(plan=plan, **kw)
    base = mqo.lib().mqo_workspace_size(dg.struct, ctypes.byref(mqo.make_params(**dict(kw, plan="batched"))), 0)
    full = mqo.lib().mqo_workspace_size(dg.struct, ctypes.byref(p), 0)
    assert base < full
    guard = 4096
    for nbytes in (base, full - 256, full):
        ws = torch.full((full + guard,), 0x5A, dtype=torch.uint8, device="cuda:0")
        bx = torch.empty(dg.n, dtype=torch.int8, device="cuda:0")
        bv = torch.empty(2, dtype=torch.int64, device="cuda:0")
        tv = torch.empty(2 * 6, dtype=torch.int64, device="cuda:0")
        r = mqo._Result(bx.data_ptr(), bv.data_ptr(), tv.data_ptr(), None)
        for _ in range(2):  # tuned, then from the cache
            assert mqo.lib().mqo_solve_mis(dg.struct, ctypes.byref(p), None, ctypes.byref(r),
                                           ctypes.c_void_p(ws.data_ptr()), nbytes, mqo._stream(dg.device)) == 0
            assert torch.equal(bv, ref["best_value"]) and torch.equal(tv, ref["traj_best_value"])
            assert torch.equal(bx, ref["best_x"])
            assert bool((ws[nbytes:] == 0x5A).all())  # nothing past what the call was given
    assert mqo.lib().mqo_solve_mis(dg.struct, ctypes.byref(p), None, ctypes.byref(r),
                                   ctypes.c_void_p(ws.data_ptr()), base - 1, mqo._stream(dg.device)) != 0
    mqo.lib().mqo_clear_caches()

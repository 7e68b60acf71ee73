"""The persistent plan's sliced-adjacency step loop (one lane per row, T = 1,
2 or 4 trajectories), forced through a tuning-cache entry, bit-exact against
the oracle: rows at the edges of the 64-row slices and of the 8-entry
blocks, a hub row, isolated rows, ragged batches, early exit and momentum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402
from oracle import solver  # noqa: E402

DEV = "cuda:0"
ELL = 2  # the sb field of a cached tile shape


@pytest.fixture(scope="module")
def mqo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo as m
    return m


def solve_with_shape(mqo, tmp_path, shape, kind, dg, **kw):
    """Solve with the persistent plan's tuned shape replaced by `shape`
    (T threads vec csr dreg ipt sb)."""
    lib, path = mqo.lib(), str(tmp_path / "tune")
    lib.mqo_clear_caches()
    mqo.solve(kind, dg, plan="persistent", **kw)
    mqo.tune_cache_save(path)
    with open(path) as f:
        lines = [ln.rstrip("\n").split("\t") for ln in f]
    key, = [k for k, v in (x for x in lines if len(x) == 2) if k.startswith("tile|")]
    value = " ".join(map(str, shape)) + " 0.001000"
    with open(path, "w") as f:
        f.writelines(ln[0] + "\n" for ln in lines if len(ln) != 2)
        f.write(f"{key}\t{value}\n")
    lib.mqo_clear_caches()
    mqo.tune_cache_load(path)
    out = mqo.solve(kind, dg, plan="persistent", **kw)
    mqo.tune_cache_save(path)
    with open(path) as f:
        assert f"{key}\t{value}" in f.read()  # feasible: not tuned again
    lib.mqo_clear_caches()
    return out


CASES = {
    "er_n64": ("mis", graphs.erdos_renyi(64, 0.3, 41)),
    "er_n65_cut": ("maxcut", graphs.erdos_renyi(65, 0.12, 42)),
    "star_and_isolated": ("maxcut", graphs.concat([graphs.star(129), graphs.empty(3), graphs.path(2)])),
    "ragged": ("mis", graphs.concat([graphs.erdos_renyi(130, 0.2, 43), graphs.cycle(17), graphs.empty(1),
                                     graphs.erdos_renyi(63, 0.5, 44), graphs.complete(9)])),
    "n700": ("maxcut", graphs.erdos_renyi(700, 0.05, 45)),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("T,threads", [(1, 256), (2, 512), (4, 1024)])
@pytest.mark.parametrize("momentum,check", [(0.0, 0), (0.4, 7)])
def test_sliced_adjacency_agrees(mqo, tmp_path, name, T, threads, momentum, check):
    kind, g = CASES[name]
    kw = dict(batch=6, steps_per_round=25, rounds=3, alpha=0.02, rho=0.1, seed=8, check_every=check)
    out = solve_with_shape(mqo, tmp_path, (T, threads, T, 0, 0, 0, ELL), kind, mqo.DeviceGraph(g, DEV),
                           momentum=momentum, **kw)
    assert out["tile_cols"] == T and out["tile_threads"] == threads and out["tile_sb"] == 0
    o = solver.solve(kind, g, solver.Params(mu=momentum, **kw))
    for key in ("traj_best_value", "traj_best_x", "best_value"):
        assert np.array_equal(out[key].cpu().numpy(), o[key]), key
    nnz_g = np.diff(g.row_ptr[g.vtx_offset])
    assert out["edge_updates"] == int((o["traj_steps"].reshape(g.num_graphs, -1) * nnz_g[:, None]).sum())


WIDE = 3


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("T,threads", [(16, 1024), (32, 1024), (32, 512), (64, 1024)])
@pytest.mark.parametrize("momentum,check", [(0.0, 0), (0.4, 7)])
def test_wide_slices_agree(mqo, tmp_path, name, T, threads, momentum, check):
    """The single-buffered step on slices of 16, 8 or 4 rows (rows paired by
    their neighbours' LDS halves at T = 32), partial last slices, unused
    columns of the tile."""
    kind, g = CASES[name]
    if max(np.diff(g.vtx_offset)) * T > 8 * 4 * threads:
        pytest.skip("more items than a thread holds")
    kw = dict(batch=37, steps_per_round=25, rounds=3, alpha=0.02, rho=0.1, seed=9, check_every=check)
    out = solve_with_shape(mqo, tmp_path, (T, threads, 4, 0, 0, 0, WIDE), kind, mqo.DeviceGraph(g, DEV),
                           momentum=momentum, **kw)
    assert out["tile_cols"] == T and out["tile_sb"] == 1
    o = solver.solve(kind, g, solver.Params(mu=momentum, **kw))
    for key in ("traj_best_value", "traj_best_x", "best_value"):
        assert np.array_equal(out[key].cpu().numpy(), o[key]), key

"""The wide slices (single-buffered tiles of 16, 32 or 64 trajectories) up to
the largest graph of every width, forced through a tuning-cache entry, bit
exact against the oracle: rows past the width whose rows are paired, a hub as
row 0 and as the last row, and automatic solves of several such graphs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402
from oracle import solver  # noqa: E402
from test_gpu_tile_ell import WIDE, solve_with_shape  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module")
def mqo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo as m
    return m


def hub_graph(n, hub, seed):
    """A random graph of mean degree about 6 with row `hub` joined to all others."""
    ru, rv, _ = graphs.erdos_renyi(n, 6.0 / n, seed).edges()
    others = np.array([v for v in range(n) if v != hub])
    return graphs.from_edges(n, np.concatenate([ru, np.full(n - 1, hub)]), np.concatenate([rv, others]))


def agrees(out, kind, g, kw):
    o = solver.solve(kind, g, solver.Params(**kw))
    for key in ("traj_best_value", "traj_best_x", "best_value"):
        assert np.array_equal(out[key].cpu().numpy(), o[key]), key


ROWS = [(16, 1024), (16, 1025), (16, 1153), (16, 1229), (16, 1500), (16, 2047), (16, 2048),
        (32, 1023), (32, 1024), (64, 509), (64, 510), (64, 511), (64, 512)]


@pytest.mark.parametrize("T,n", ROWS)
@pytest.mark.parametrize("kind,shape", [("mis", "er"), ("maxcut", "hub_first"), ("mis", "hub_last")])
def test_wide_slices_of_large_graphs_agree(mqo, tmp_path, T, n, kind, shape):
    g = (graphs.erdos_renyi(n, 24.0 / n, 50 + n) if shape == "er" else
         hub_graph(n, 0 if shape == "hub_first" else n - 1, 60 + n))
    kw = dict(batch=T + 3, steps_per_round=15, rounds=2, alpha=0.02, rho=0.1, seed=n)
    out = solve_with_shape(mqo, tmp_path, (T, 1024, 4, 0, 0, 0, WIDE), kind, mqo.DeviceGraph(g, DEV), **kw)
    assert out["tile_cols"] == T and out["tile_sb"] == 1
    agrees(out, kind, g, kw)


@pytest.mark.parametrize("plan", ["persistent", "auto"])
def test_batch_of_large_graphs_agrees(mqo, plan):
    g = graphs.concat([graphs.erdos_renyi(1500, 0.016, 71), graphs.barabasi_albert(1400, 4, 72),
                       hub_graph(1300, 0, 73), graphs.erdos_renyi(1537, 0.01, 74)])
    kw = dict(batch=130, steps_per_round=12, rounds=2, alpha=0.02, rho=0.1, seed=3)
    mqo.lib().mqo_clear_caches()
    out = mqo.solve("mis", mqo.DeviceGraph(g, DEV), plan=plan, **kw)
    mqo.lib().mqo_clear_caches()
    agrees(out, "mis", g, kw)

"""Persistent solves at the edge of the LDS: graphs whose tile of 2, 4, 8 or
16 trajectories fits beside the kernel's own arrays by a little or misses by a
little.  Shapes that miss are not offered, and no failed launch is reported by
the next one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402
from oracle import solver  # noqa: E402

DEV = "cuda:0"

# one or two iterate tiles, row_ptr and the row order: (4 or 8) T + 6 bytes a
# row in 163 840 less the static arrays' 3600; a single buffer of 4
# trajectories is the widest that many rows allow
SIZES = sorted({(T, 160240 // (bytes_row + 6) + d) for T, bytes_row in ((2, 16), (3, 16), (4, 32), (8, 64))
                for d in (-3, -1, 0, 1, 5, 18, 45)})


@pytest.mark.parametrize("T,n", SIZES)
@pytest.mark.parametrize("weighted", [True, False])
def test_solves_at_the_edge_of_the_lds(T, n, weighted):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    g = graphs.erdos_renyi(n, 3.0 / n, n)
    if weighted:
        g = graphs.with_weights(g, 5, (-2, 1, 3))
    kw = dict(batch=T, steps_per_round=4, rounds=2, alpha=0.02, rho=0.1, seed=7)
    mqo.lib().mqo_clear_caches()
    out = mqo.solve("maxcut", mqo.DeviceGraph(g, DEV), plan="persistent", **kw)
    mqo.lib().mqo_clear_caches()
    o = solver.solve("maxcut", g, solver.Params(**kw))
    for key in ("traj_best_value", "traj_best_x", "best_value"):
        assert np.array_equal(out[key].cpu().numpy(), o[key]), key

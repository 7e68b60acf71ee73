"""OneTwoSwap on dense graphs, where the pair iterations after the first work
only on the columns that moved, and the priorities of many graphs are drawn in
shared launches: against the oracle for a ragged batch of more graphs than a
launch's table takes, with column counts around the 64-column words."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import discrete  # noqa: E402
from synth import graphs  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module")
def mqo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo as m
    return m


@pytest.mark.parametrize("B", [1, 64, 65, 200])
def test_live_columns_equal_each_graph(mqo, B):
    rng = np.random.default_rng(61)
    gs = [graphs.erdos_renyi(int(n), 0.4, 400 + i) for i, n in enumerate(rng.integers(50, 150, 67))]
    g = graphs.concat(gs)
    assert g.nnz / g.n >= 24  # the searches with a wavefront per row
    dg = mqo.DeviceGraph(g, DEV)
    Z = mqo.round_evaluate("mis", dg, mqo.init_iterate("mis", dg, B, 62))[0]
    start = Z.cpu().numpy()
    mqo.pair_search("mis", dg, Z, 62, 3)
    got = Z.cpu().numpy()
    # sampled graphs (first, last of the first table, first of the second) on
    # the oracle, a few columns each
    for gi in (0, 63, 64, 66):
        lo, hi = int(g.vtx_offset[gi]), int(g.vtx_offset[gi + 1])
        cols = np.array(sorted({0, B // 2, B - 1}))
        ref, _ = discrete.pair_search("mis", gs[gi], start[lo:hi][:, cols], 62, gi * B + cols, 3)
        assert np.array_equal(got[lo:hi][:, cols], ref), gi

"""The unrolled adjoint over segments of every length: the states and masks of
a step do not depend on where the checkpoints lie, so dL/dx_0 is the same bit
for bit for every ckpt_every, and dL/dalpha to the rounding of its float64
sums; a segment of one step (whose only step is its last) against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import pga  # noqa: E402
from synth import graphs  # noqa: E402

DEV = "cuda:0"
K = 12
CASES = {
    "regular": ("maxcut", graphs.random_regular(600, 5, 1), 8),
    "hubs": ("mis", graphs.barabasi_albert(900, 4, 2), 5),
    "weighted": ("maxcut", graphs.torus_pm1(17, 3), 6),
    "batch": ("mis", graphs.concat([graphs.erdos_renyi(90, 0.1, 4), graphs.star(40), graphs.erdos_renyi(33, 0.3, 5)]), 4),
}


@pytest.mark.parametrize("name", list(CASES))
def test_segments_of_every_length_agree(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    kind, g, B = CASES[name]
    param, alpha = (2.0, 0.05) if kind == "mis" else (1e-3, 0.05)
    dg = mqo.DeviceGraph(g, DEV, hub_min_degree=40)
    rng = np.random.default_rng(7)
    lo = 0.0 if kind == "mis" else -1.0
    x0 = rng.uniform(lo, 1.0, (g.n, B)).astype(np.float32)
    dL = rng.standard_normal((g.n, B)).astype(np.float32)
    ref = None
    for c in (1, 2, 3, 4, 6, 12):
        XK, ck = mqo.unrolled_forward(kind, dg, torch.from_numpy(x0).to(DEV), alpha, K, c, param)
        top = torch.from_numpy(dL).to(DEV)
        dX, da = mqo.unrolled_backward(kind, dg, ck, top, alpha, K, c, param)
        assert torch.equal(top, torch.from_numpy(dL).to(DEV))
        if ref is None:
            ref = dX, da
            rX, ra = pga.unrolled_backward(g, kind, param, alpha, K, x0, dL.astype(np.float64), precision="fp32")
            assert np.allclose(dX.cpu().numpy(), rX, rtol=1e-4, atol=1e-4 * np.abs(rX).max())
            if g.num_graphs == 1:
                assert np.allclose(da.cpu().numpy(), ra, rtol=1e-4, atol=1e-4 * np.abs(ra).max())
        assert torch.equal(dX, ref[0]), c
        # float64 sums of at most n K terms in another order
        scale = g.n * K * 2.0 ** -53 * max(1.0, float(ref[1].abs().max())) * 16
        assert torch.allclose(da, ref[1], rtol=0.0, atol=scale), c

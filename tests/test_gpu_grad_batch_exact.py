"""Objective values of a batch against each graph on its own, bit for bit:
graphs whose rows are grouped alike in both (none near-regular), with partial
sums that take one level and two."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("kind,param,B", [("mis", 2.0, 32), ("maxcut", 1e-3, 7), ("maxcut_fl", 0.0, 64)])
def test_values_equal_each_graphs_own(kind, param, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    gs = [graphs.erdos_renyi(n, 6.0 / n, 400 + i) for i, n in enumerate((9, 4000, 77, 300, 2500, 40, 1000))]
    g = graphs.concat(gs)
    dg = mqo.DeviceGraph(g, DEV, hub_min_degree=None)
    X = torch.rand(g.n, B, generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    f, grad = mqo.objective_grad(kind, dg, X, param)
    for i, sub in enumerate(gs):
        lo, hi = int(g.vtx_offset[i]), int(g.vtx_offset[i + 1])
        fi, gi = mqo.objective_grad(kind, mqo.DeviceGraph(sub, DEV, hub_min_degree=None), X[lo:hi].contiguous(), param)
        assert torch.equal(f[i * B:(i + 1) * B], fi) and torch.equal(grad[lo:hi], gi), i

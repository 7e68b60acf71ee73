"""Objective and gradient of a batch of graphs in shared launches: bit for bit
the values of each graph on its own (more graphs than a launch's table takes,
graphs whose partial sums go through slices, odd column counts, weights,
every formulation, the smallest workspace), and the backward that scales the
forward's gradient against the one that runs the product again."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module")
def mqo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo as m
    return m


def _batch(many):
    rng = np.random.default_rng(31)
    gs = [graphs.erdos_renyi(int(n), 0.1, 300 + i) for i, n in enumerate(rng.integers(1, 90, 70 if many else 3))]
    return gs + [graphs.random_regular(4000, 3, 33), graphs.empty(2), graphs.cycle(2500)]


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("kind,param,weighted,B", [("mis", 2.0, False, 32), ("maxcut", 1e-3, False, 7),
                                                   ("maxcut", 1e-3, True, 64), ("maxcut_fp", 0.5, True, 10),
                                                   ("maxcut_fl", 0.0, False, 1), ("maxcut_fa", 0.0, True, 130)])
def test_batch_equals_each_graph(mqo, many, kind, param, weighted, B):
    gs = _batch(many)
    if weighted:
        gs = [graphs.with_weights(g, 40 + i) for i, g in enumerate(gs)]
    g = graphs.concat(gs)
    dg = mqo.DeviceGraph(g, DEV, hub_min_degree=None)
    gen = torch.Generator(device=DEV).manual_seed(5)
    X = torch.rand(g.n, B, generator=gen, device=DEV) * 2 - 1
    scale = torch.randn(g.num_graphs * B, generator=gen, device=DEV)
    f, grad = mqo.objective_grad(kind, dg, X, param, scale=scale)
    _, grad1 = mqo.objective_grad(kind, dg, X, param, want_f=False)
    # the smallest workspace that is taken: few graphs per launch
    lib = mqo.lib()
    big = max(gs, key=lambda x: x.n)
    need = lib.mqo_objective_workspace_size(mqo.DeviceGraph(big, DEV, hub_min_degree=None).struct, B)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    f2 = torch.empty_like(f)
    k = mqo._KIND[kind]
    status = lib.mqo_objective_grad(dg.struct, k, param, ctypes.c_void_p(X.data_ptr()), B, None,
                                    ctypes.c_void_p(f2.data_ptr()), None, ctypes.c_void_p(ws.data_ptr()), need,
                                    mqo._stream(DEV))
    assert status == 0 and torch.equal(f2, f)
    for i, sub in enumerate(gs):
        lo, hi = int(g.vtx_offset[i]), int(g.vtx_offset[i + 1])
        dsub = mqo.DeviceGraph(sub, DEV, hub_min_degree=None)
        dsub._struct.max_degree = dg.max_degree  # the batch's near-regular test
        fi, gi = mqo.objective_grad(kind, dsub, X[lo:hi].contiguous(), param,
                                    scale=scale[i * B:(i + 1) * B].contiguous())
        assert torch.equal(grad[lo:hi], gi), i
        assert torch.allclose(f[i * B:(i + 1) * B], fi, rtol=1e-12, atol=1e-12 * max(1, sub.n)), i
        _, gi = mqo.objective_grad(kind, dsub, X[lo:hi].contiguous(), param, want_f=False)
        assert torch.equal(grad1[lo:hi], gi), i


@pytest.mark.parametrize("B", [32, 7])
@pytest.mark.parametrize("hubs", [False, True])
def test_backward_scales_the_forward_gradient(mqo, B, hubs):
    g = graphs.barabasi_albert(3000, 4, 51) if hubs else graphs.concat(_batch(True))
    dg = mqo.DeviceGraph(g, DEV)
    gen = torch.Generator(device=DEV).manual_seed(6)
    X = torch.rand(g.n, B, generator=gen, device=DEV).requires_grad_(True)
    up = torch.randn(g.num_graphs * B, generator=gen, device=DEV, dtype=torch.float64)
    f = mqo.objective(X, dg, "mis", 2.0)
    f.backward(up)
    f0, ref = mqo.objective_grad("mis", dg, X.detach(), 2.0, scale=up)
    assert torch.equal(f.detach(), f0) and torch.equal(X.grad, ref)
    # an expanded upstream gradient, a strided X, no gradient asked for
    X.grad = None
    mqo.objective(X, dg, "mis", 2.0).sum().backward()
    assert torch.equal(X.grad, mqo.objective_grad("mis", dg, X.detach(), 2.0)[1])
    assert not mqo.objective(X.detach(), dg, "mis", 2.0).requires_grad
    with torch.no_grad():
        assert torch.equal(mqo.objective(X.detach().t().contiguous().t(), dg, "mis", 2.0), f0)
    # a change to X between forward and backward is refused
    f = mqo.objective(X, dg, "mis", 2.0)
    with torch.no_grad():
        X.mul_(0.5)
    with pytest.raises(RuntimeError):
        f.backward(up)

"""The gradient that an Objective's forward keeps: one more array like X until
the backward has run, and none where it is larger than the share of the GPU's
memory that it may take; the gradient is the same in both cases."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("kind,param", [("mis", 2.0), ("maxcut", 1e-3)])
def test_large_gradients_are_not_kept(monkeypatch, kind, param):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    assert mqo._kept_gradient_bytes(torch.device(DEV)) == torch.cuda.get_device_properties(DEV).total_memory // 16
    dg = mqo.DeviceGraph(graphs.erdos_renyi(40000, 2e-4, 1), DEV)
    X = torch.rand(dg.n, 64, device=DEV, requires_grad=True)
    nbytes, grads = 4 * X.numel(), []
    w = torch.rand(64, dtype=torch.float64, device=DEV)
    for room in (nbytes, nbytes - 1):
        monkeypatch.setattr(mqo, "_kept_gradient_bytes", lambda device: room)
        mqo.objective(X, dg, kind, param).sum()  # the workspace is there
        before = torch.cuda.memory_allocated()
        f = mqo.objective(X, dg, kind, param)
        kept = torch.cuda.memory_allocated() - before
        assert (kept >= nbytes) == (room >= nbytes)
        grads.append(torch.autograd.grad((f * w).sum(), X)[0])
        del f
    assert torch.equal(grads[0], grads[1])

"""The auto plan's trial of both plans on a workspace that holds whatever was
in memory: the persistent trial's error word is cleared before it runs.  The
trial runs when the tuned times of the two plans lie within a factor of two,
so the tile shape's cached time is swept in steps of 1.5."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import solver  # noqa: E402
from synth import graphs  # noqa: E402

DEV = "cuda:0"


def test_trial_on_a_dirty_workspace(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    lib, path = mqo.lib(), str(tmp_path / "tune")
    g = graphs.erdos_renyi(150, 0.1, 71)
    dg = mqo.DeviceGraph(g, DEV)
    kw = dict(batch=8, steps_per_round=20, rounds=3, alpha=0.02, rho=0.1, seed=9)
    o = solver.solve("mis", g, solver.Params(**kw))
    ws = mqo.Workspace(DEV)
    lib.mqo_clear_caches()
    mqo.solve("mis", dg, plan="persistent", workspace=ws, **kw)
    mqo.tune_cache_save(path)
    with open(path) as f:
        lines = [ln.rstrip("\n").split("\t") for ln in f]
    (key, value), = [ln for ln in lines if len(ln) == 2 and ln[0].startswith("tile|")]
    trials = 0
    for i in range(15):
        with open(path, "w") as f:
            f.writelines(ln[0] + "\n" for ln in lines if len(ln) != 2)
            f.write(f"{key}\t{' '.join(value.split()[:-1])} {0.0005 * 1.5 ** i:.6f}\n")
        lib.mqo_clear_caches()
        mqo.tune_cache_load(path)
        ws.buf.fill_(0xFF)
        out = mqo.solve("mis", dg, plan="auto", workspace=ws, **kw)
        for name in ("traj_best_value", "traj_best_x", "best_value"):
            assert np.array_equal(out[name].cpu().numpy(), o[name]), name
        mqo.tune_cache_save(path)
        with open(path) as f:
            plan, = [ln.split("\t")[1] for ln in f if ln.startswith("plan|")]
        trials += float(plan.split()[3]) > 0.0
    lib.mqo_clear_caches()
    assert trials > 0

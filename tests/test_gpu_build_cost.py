"""A sliced shape is taken where its steps earn its build back: the tuning
cache holds the build's time and the fastest shape without one beside the
fastest per step, and every solve weighs the two by its own steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import solver  # noqa: E402
from synth import graphs  # noqa: E402

DEV = "cuda:0"
SLICED, PLAIN = "2 512 2 0 0 0 2", "8 1024 2 0 0 0 0"


def test_the_build_is_weighed_by_the_steps_of_the_solve(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    lib, path = mqo.lib(), str(tmp_path / "tune")
    g = graphs.erdos_renyi(200, 0.1, 91)
    dg = mqo.DeviceGraph(g, DEV)
    kw = dict(batch=8, alpha=0.02, rho=0.1, seed=9, plan="persistent")
    lib.mqo_clear_caches()
    mqo.solve("mis", dg, steps_per_round=40, rounds=1, **kw)
    mqo.tune_cache_save(path)
    with open(path) as f:
        key, = [ln.split("\t")[0] for ln in f if ln.startswith("tile|")]
    # 1 us and 3 us a step, a build of 200 us: even at 100 steps
    with open(path, "w") as f:
        f.write(f"{key}\t{SLICED} 0.001000\nbuild|{key[5:]}\t0.200000 {PLAIN} 0.003000\n")
    for steps, rounds, T in ((99, 1, 8), (101, 1, 2), (0, 1, 8), (20, 4, 8), (20, 6, 2)):
        lib.mqo_clear_caches()
        mqo.tune_cache_load(path)
        out = mqo.solve("mis", dg, steps_per_round=steps, rounds=rounds, **kw)
        assert out["tile_cols"] == T, (steps, rounds)
        o = solver.solve("mis", g, solver.Params(batch=8, alpha=0.02, rho=0.1, seed=9, steps_per_round=steps,
                                                 rounds=rounds))
        for name in ("traj_best_value", "traj_best_x", "best_value"):
            assert np.array_equal(out[name].cpu().numpy(), o[name]), name
    # without the second entry, or with one that does not parse, the first is taken as it is
    for line in ("", f"build|{key[5:]}\t0.200000 nothing\n"):
        with open(path, "w") as f:
            f.write(f"{key}\t{SLICED} 0.001000\n{line}")
        lib.mqo_clear_caches()
        mqo.tune_cache_load(path)
        assert mqo.solve("mis", dg, steps_per_round=5, rounds=1, **kw)["tile_cols"] == 2
    lib.mqo_clear_caches()

"""Automatic solves of few short steps: the plan is timed on the whole solve,
not on its steps alone, and the choice is cached apart from the one of longer
rounds (n = 3000, degree 100: the persistent step is four times as fast, but a
solve of one round of 10 steps is not)."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402

DEV = "cuda:0"


def solve_ms(mqo, dg, **kw):
    ts = []
    for i in range(12):
        torch.cuda.synchronize()
        t = time.perf_counter()
        mqo.solve("mis", dg, **kw)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return 1e3 * float(np.median(ts[2:]))


def test_short_and_long_rounds_choose_apart(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    lib, path = mqo.lib(), str(tmp_path / "tune")
    dg = mqo.DeviceGraph(graphs.erdos_renyi(3000, 100 / 2999, 4), DEV)
    kw = dict(batch=64, alpha=0.02, rho=0.1, seed=1)
    lib.mqo_clear_caches()
    long = mqo.solve("mis", dg, steps_per_round=200, rounds=2, **kw)
    short = dict(steps_per_round=10, rounds=1, **kw)
    chosen = mqo.solve("mis", dg, **short)["plan"]
    each = {plan: solve_ms(mqo, dg, plan=plan, **short) for plan in ("persistent", "batched")}
    mqo.tune_cache_save(path)
    lib.mqo_clear_caches()
    with open(path) as f:
        plans = [ln.split("\t") for ln in f if ln.startswith("plan|")]
    assert len(plans) == 2 and plans[0][0] != plans[1][0]
    assert long["plan"] == "persistent"
    # the chosen plan is the better one (they are a quarter apart), or as good
    assert each[chosen] <= 1.1 * min(each.values()), (chosen, each)

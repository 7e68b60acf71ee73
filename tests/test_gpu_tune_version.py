"""Tuning-cache entries written before the tile keys carried a version (their
times may be of slices that held one row only) are not taken: the shape is
tuned again, and the old lines stay in the file as they are."""
import re

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import graphs  # noqa: E402

DEV = "cuda:0"


def entries(path):
    with open(path) as f:
        return dict(ln.rstrip("\n").split("\t") for ln in f if "\t" in ln)


@pytest.mark.parametrize("plan", ["persistent", "auto"])
def test_entries_without_a_version_are_not_taken(tmp_path, plan):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    lib, path = mqo.lib(), str(tmp_path / "tune")
    dg = mqo.DeviceGraph(graphs.erdos_renyi(150, 0.1, 81), DEV)
    kw = dict(batch=8, steps_per_round=20, rounds=2, alpha=0.02, rho=0.1, seed=9, plan=plan)
    lib.mqo_clear_caches()
    mqo.solve("mis", dg, **kw)
    mqo.tune_cache_save(path)
    old = {}
    for key in entries(path):
        kind, rest = key.split("|", 1)
        if kind not in ("tile", "plan"):
            continue
        rest = re.sub(r"\|v\d+\|", "|", rest, count=1)
        # a shape that the tuner would not leave alone: one trajectory of 64
        # trajectories' room; a plan that is not the tuner's
        old[f"{kind}|{rest}"] = "64 256 1 0 0 0 0 0.000001" if kind == "tile" else "batched 1.0 0.1 -1.0 -1.0"
    with open(path, "w") as f:
        f.writelines(f"{k}\t{v}\n" for k, v in old.items())
    lib.mqo_clear_caches()
    mqo.tune_cache_load(path)
    out = mqo.solve("mis", dg, **kw)
    mqo.tune_cache_save(path)
    got = entries(path)
    lib.mqo_clear_caches()
    assert out["tile_cols"] < 64 and out["plan"] == "persistent"
    for key, value in old.items():
        assert got[key] == value and len([k for k in got if k.startswith(key.split("|")[0] + "|")]) == 2

"""What a tuned shape is reused for: the same jet, and no jet whose fastest
shape differs from it by the library's own measurements (another grid of the
same size class, equilibrium sides, a wall at column -1, a table beyond LDS, or
another set of compiled shapes).  The timing is replaced by a table, so no GPU
is needed."""
import json
import os

import numpy as np
import pytest

from gpu_common import tiny_params


@pytest.fixture
def tuner(tmp_path, monkeypatch):
    from paper_1002_3028_amd import autotune, build, lbm
    if not os.path.exists(lbm.LIB_PATH):
        build.build()
    monkeypatch.setenv("LBM_AUTOTUNE_CACHE", str(tmp_path / "autotune.json"))
    monkeypatch.setattr(autotune, "_arch", lambda: "gfx950")
    calls = []

    def timed(params, inlet, precision, shapes=None, **kw):
        n = len(lbm.tile_shapes())
        order = list(range(n) if shapes is None else shapes)
        calls.append((params["nx"], params["nr"]))
        best = order[len(calls) % len(order)]  # each timing finds another shape fastest
        return {q: 1e-6 if q == best else 2e-6 for q in order}

    monkeypatch.setattr(autotune, "time_shapes", timed)
    return autotune, lbm, calls, tmp_path / "autotune.json"


def _jet(nx, nr, case="jet", table=None):
    p = tiny_params(nx, nr, case, 1)
    if table:
        p["nu_mult"], p["alpha_mult"] = np.linspace(1, 8, table), np.linspace(1, 20, table)
    return p


def test_each_jet_is_timed_once(tuner):
    autotune, _, calls, _ = tuner
    first = autotune.best_shape(_jet(128, 32), None, "fp32")
    assert autotune.best_shape(_jet(128, 32), None, "fp32") == first and len(calls) == 1
    # a table in LDS and edges that cost nothing extra do not matter
    assert autotune.best_shape(_jet(128, 32, table=200), None, "fp32") == first
    assert autotune.best_shape(_jet(128, 32, "slab"), None, "fp32") == first and len(calls) == 1


@pytest.mark.parametrize("other", [
    dict(nx=400, nr=300), dict(nx=128, nr=33), dict(case="eq"), dict(case="xwalls"),
    dict(case="closed"), dict(table=300)], ids=str)
def test_other_jets_are_timed_themselves(tuner, other):
    autotune, _, calls, _ = tuner
    first = autotune.best_shape(_jet(128, 32), None, "fp32")
    got = autotune.best_shape(_jet(**{**dict(nx=128, nr=32), **other}), None, "fp32")
    assert len(calls) == 2 and got != first


def test_results_of_other_shape_sets_are_not_reused(tuner, monkeypatch):
    autotune, lbm, calls, cache = tuner
    p = _jet(2048, 512)
    # an entry as earlier versions wrote it
    cls = autotune.size_class(lbm.bytes_required(p, "fp32"))
    cache.write_text(json.dumps({f"gfx950/fp32/{cls}": {"info": lbm.tile_shape_info(23),
                                                        "s_per_step": 1e-9}}))
    autotune.best_shape(p, None, "fp32")
    assert len(calls) == 1
    infos = lbm.tile_shape_infos()
    monkeypatch.setattr(lbm, "tile_shape_infos", lambda: infos[:-1])
    autotune.best_shape(p, None, "fp32")
    assert len(calls) == 2


def test_batch_key_tells_edges_and_tables_apart(tuner):
    autotune = tuner[0]
    sets = [[_jet(128, 32)] * 4, [_jet(128, 32)] * 3 + [_jet(128, 32, "eq")],
            [_jet(128, 32)] * 3 + [_jet(128, 32, table=300)]]
    keys = [autotune.batch_key([(p, None) for p in s], "fp32") for s in sets]
    assert len(set(keys)) == 3

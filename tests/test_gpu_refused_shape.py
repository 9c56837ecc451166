"""A refused lbm_set_tile_shape (an index that does not exist, or any shape but
0 on a single buffer) leaves the run as it was: the steps after it are, bit for
bit, those of a run without the call, also where directly launched steps have
left the device's descriptor behind the step count."""
import numpy as np
import pytest

from gpu_common import noisy_inlet, require_gpu, tiny_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 6, 7])
@pytest.mark.parametrize("kw", [dict(tile_shape=0), dict(), dict(graph_steps=4),
                                dict(layout="single")], ids=str)
def test_refused_shape_changes_nothing(kw, steps):
    require_gpu()
    from paper_1002_3028_amd import lbm
    p = tiny_params(130, 33, "jet", 1)
    n = len(lbm.tile_shapes())
    out = []
    for refuse in (False, True):
        with lbm.Solver(p, "fp16sr", **kw) as s:
            s.set_inlet(*noisy_inlet(33, 5, 3))
            s.step(steps)
            for q in ((-1, n, 5) if kw.get("layout") else (-1, n)) if refuse else ():
                with pytest.raises(lbm.LbmError) as e:
                    s.set_tile_shape(q)
                assert e.value.code == lbm.EINVAL
            s.step(steps)
            out.append((s.step_count,) + s.get_populations())
    assert out[0][0] == out[1][0] == 2 * steps
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][2], out[1][2])

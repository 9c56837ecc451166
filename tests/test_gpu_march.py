"""Several time steps per launch with the intermediate states in registers
(marching waves, and stacked rows on small grids): bit-identical to one-step launches (shape 0) on every edge
rule and storage form, at strips and tiles that end one node off an edge of
the domain, on grids narrower than a strip or its halo, for step counts with
a remainder, with property tables that fit LDS and tables that do not, and in
a batch whose jets stop inside a launch.
"""
import numpy as np
import pytest

from gpu_common import CASES, noisy_inlet, require_gpu, tiny_params

pytestmark = pytest.mark.gpu

# (nx, nr): one strip (58 columns marching; 58, 56, 54 or 50 stacked) and a
# column more or less; several strips; narrower than the halo; the fewest
# rows; tiles (stacked: 10, 8, 6 or 2 rows) that end on, before and after the
# last row
GRIDS = [(58, 16), (59, 17), (57, 2), (50, 10), (56, 11), (55, 7), (200, 45), (2, 3), (5, 9),
         (175, 130)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _march_shapes():
    from paper_1002_3028_amd import lbm
    return [q for q, inf in enumerate(lbm.tile_shape_infos()) if inf["steps"] > 2]


def _state(p, inlet, steps, precision, **kw):
    from paper_1002_3028_amd import inputs, lbm
    with lbm.Solver(p, precision, **kw) as s:
        s.set_state(*inputs.perturbed_state(p["nx"], p["nr"], seed=p["nx"] + 7 * p["nr"],
                                            noise=0.3))
        if inlet is not None:
            s.set_inlet(*inlet)
        s.step(steps)
        f, g = s.get_populations()
        return f, g, s.moments()  # (moments read the ghost ring too)


def _same(a, b, what):
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), what
    for k in a[2]:
        assert np.array_equal(a[2][k], b[2][k]), (what, k)


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16", "fp16sr"])
@pytest.mark.parametrize("case", CASES)
def test_march_equals_single(case, precision):
    shapes = _march_shapes()
    assert shapes
    for nx, nr in GRIDS:
        p = tiny_params(nx, nr, case, (nx + nr) % 2)
        inlet = noisy_inlet(nr, 5, nx) if p["bc"][0] == "inlet" else None
        ref = _state(p, inlet, 23, precision, tile_shape=0)
        for q in shapes:
            for gk in (0, 10):
                got = _state(p, inlet, 23, precision, tile_shape=q, graph_steps=gk)
                _same(got, ref, (case, precision, nx, nr, q, gk))


def test_march_large_table_and_none():
    """Property tables of 2, 256, 257 and 1000 entries and constant
    properties: the table in LDS and the table in memory give the same bits."""
    for n in (0, 2, 256, 257, 1000):
        p = tiny_params(130, 40, "jet", 1)
        if n == 0:
            p["nu_mult"] = p["alpha_mult"] = None
        else:
            p["nu_mult"] = np.linspace(1.0, 8.0, n)
            p["alpha_mult"] = np.linspace(1.0, 20.0, n)
        inlet = noisy_inlet(40, 4, 1)
        ref = _state(p, inlet, 21, "fp32", tile_shape=0)
        for q in _march_shapes():
            _same(_state(p, inlet, 21, "fp32", tile_shape=q), ref, (n, q))


@pytest.mark.parametrize("precision", ["fp32", "fp16sr"])
def test_batch_march_with_uneven_targets(precision):
    """Jets whose targets leave every remainder of a launch, in groups of 10,
    7 and 3 steps, one with a property table beyond LDS: each equals itself
    alone with one step per launch."""
    from paper_1002_3028_amd import lbm
    jets = []
    for q, (nx, nr, case, steps) in enumerate([(200, 45, "jet", 61), (64, 16, "xwalls", 62),
                                                (130, 33, "substrate", 63), (90, 20, "slab", 64),
                                                (70, 12, "closed", 65), (59, 30, "jet", 1)]):
        p = tiny_params(nx, nr, case, q % 2)
        if q == 3:
            p["nu_mult"], p["alpha_mult"] = np.linspace(1, 8, 300), np.linspace(1, 20, 300)
        jets.append((p, noisy_inlet(nr, 3 + q, q) if p["bc"][0] == "inlet" else None, steps))
    refs = []
    for p, inlet, steps in jets:
        with lbm.Batch(1 << 28, 1, precision) as alone:
            alone.set_launch(0, 0)
            s = alone.admit(p, inlet, steps)
            alone.run(steps)
            refs.append(alone.moments(s))
    for q in _march_shapes():
        for grid in (0, 8):
            with lbm.Batch(1 << 30, 8, precision) as b:
                b.set_launch(q, grid)
                slots = [b.admit(*j) for j in jets]
                for k in (10, 10, 10, 7, 7, 7, 3, 3, 3, 3, 3):
                    b.run(k)
                assert [b.poll(s) for s in slots] == [st for _, _, st in jets]
                for n, (s, r) in enumerate(zip(slots, refs)):
                    m = b.moments(s)
                    for k in r:
                        assert np.array_equal(m[k], r[k]), (q, grid, n, k)


def test_march_flags_instability():
    from paper_1002_3028_amd import inputs, lbm
    p = tiny_params(64, 16, "jet", 0)
    for q in _march_shapes():
        with lbm.Solver(p, "fp32", tile_shape=q) as s:
            s.set_inlet(*inputs.inlet_rows(16, 8.0, 0.9, 5.0))
            s.step(400)
            assert s.try_sync() == lbm.EUNSTABLE


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16", "fp16sr"])
@pytest.mark.parametrize("case", CASES)
def test_default_shape_equals_single(case, precision):
    """The shape a solver takes by itself: on a grid where it is the stacked
    rows, and on one of half a million nodes where storage form and edge rules
    decide between marching, two steps and one step per launch."""
    for nx, nr in [(600, 150), (1030, 515)]:
        p = tiny_params(nx, nr, case, 0)
        inlet = noisy_inlet(nr, 5, nx) if p["bc"][0] == "inlet" else None
        ref = _state(p, inlet, 11, precision, tile_shape=0)
        _same(_state(p, inlet, 11, precision), ref, (case, precision, nx, nr))


@pytest.mark.parametrize("streams", [1, 2, 3, 4])
def test_batch_split_over_streams(streams):
    """Jets whose buffers (52 MB) are split evenly over the streams' cohorts,
    one far larger than the rest, retired one after another until the rest is
    too little to split: each equals itself alone."""
    from paper_1002_3028_amd import lbm
    sizes = [(300, 70, 31), (1500, 200, 40), (700, 150, 52), (290, 60, 64)]
    jets = [(tiny_params(nx, nr, "jet", q % 2), noisy_inlet(nr, 3, q), n)
            for q, (nx, nr, n) in enumerate(sizes)]
    refs = []
    for p, inlet, n in jets:
        with lbm.Batch(1 << 28, 1, "fp32") as alone:
            alone.set_launch(0, 0)
            s = alone.admit(p, inlet, n)
            alone.run(n)
            refs.append(alone.moments(s))
    with lbm.Batch(1 << 28, 8, "fp32") as b:
        b.set_streams(streams)
        slots = [b.admit(*j) for j in jets]
        for _ in range(13):
            b.run(5)
        for s, r in zip(slots, refs):
            m = b.moments(s)
            for k in r:
                assert np.array_equal(m[k], r[k]), (streams, s, k)


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16", "fp16sr"])
@pytest.mark.parametrize("case", CASES)
def test_tall_tiles_and_second_filling(case, precision):
    """1030 x 515: both marching shapes take five rows a wave, so that most of
    a wave's rows have all levels active, and more workgroups (468 with four
    steps per launch, 494 with five) than the device has CUs, so that the
    waves of the second filling run too.  Launches of every step count up to
    the shape's."""
    from paper_1002_3028_amd import lbm
    nx, nr = 1030, 515
    p = tiny_params(nx, nr, case, 1)
    inlet = noisy_inlet(nr, 5, nx) if p["bc"][0] == "inlet" else None
    ref = _state(p, inlet, 13, precision, tile_shape=0)
    marching = [q for q in _march_shapes() if lbm.tile_shape_info(q)["by"] == 4]
    assert sorted(lbm.tile_shape_info(q)["steps"] for q in marching) == [4, 5]
    for q in marching:
        _same(_state(p, inlet, 13, precision, tile_shape=q), ref, (case, precision, q))
        _same(_state(p, inlet, 13, precision, tile_shape=q, graph_steps=11), ref,
              (case, precision, q, "graph"))

"""The last steps of a group, and single steps, where a solver or batch chose
its shape by itself: fewer steps than a launch holds take the shape that is
faster for them (seen by the kernels launched), in any order of step counts and
with jets that stop anywhere, bit-identical to one step per launch."""
import warnings

import numpy as np
import pytest

from gpu_common import noisy_inlet, require_gpu, tiny_params

pytestmark = pytest.mark.gpu

# one round of stacked rows; two in FP32; marching; marching with states that
# the Infinity Cache does not hold (FP32, and all forms)
GRIDS = [(128, 32), (800, 210), (1030, 515), (2620, 1000), (3310, 1600)]
COUNTS = (1, 2, 3, 4, 5, 6, 7, 9, 1, 13, 2)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _jet(nx, nr, case="jet"):
    p = tiny_params(nx, nr, case, 1)
    return p, noisy_inlet(nr, 5, nx) if p["bc"][0] == "inlet" else None


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16", "fp16sr"])
@pytest.mark.parametrize("nx,nr", GRIDS)
def test_any_counts_equal_single_steps(nx, nr, precision):
    from paper_1002_3028_amd import inputs, lbm
    p, inlet = _jet(nx, nr)
    st = inputs.perturbed_state(nx, nr, seed=nx, noise=0.3)
    out = []
    for kw in (dict(tile_shape=0), dict(), dict(graph_steps=6)):
        with lbm.Solver(p, precision, **kw) as s:
            s.set_state(*st)
            s.set_inlet(*inlet)
            for n in COUNTS:
                s.step(n)
            assert s.step_count == sum(COUNTS)
            out.append((s.moments(), s.conservation()))
    for got in out[1:]:
        assert got[1] == out[0][1]
        for k in out[0][0]:
            assert np.array_equal(got[0][k], out[0][0][k]), k


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp16sr"])
@pytest.mark.parametrize("sizes", [[(1030, 515)], [(512, 128)] * 8, [(128, 32), (200, 45)]],
                         ids=str)
def test_batch_groups_of_any_length(sizes, precision):
    """Jets that stop at every remainder of a group, in groups of 1 to 11
    steps: each equals itself alone with one step per launch."""
    from paper_1002_3028_amd import lbm
    jets = [_jet(nx, nr, "jet") + (17 + 5 * q,) for q, (nx, nr) in enumerate(sizes)]
    with lbm.Batch(1 << 28, 8, precision) as b:
        slots = [b.admit(*j) for j in jets]
        for k in (1, 2, 3, 5, 6, 7, 9, 10, 11, 1, 2, 3, 4):
            b.run(k)
        assert [b.poll(s) for s in slots] == [j[2] for j in jets]
        got = [b.moments(s) for s in slots]
    for (p, inlet, n), m in zip(jets, got):
        with lbm.Solver(p, precision, tile_shape=0) as s:
            s.set_inlet(*inlet)
            s.step(n)
            ref = s.moments()
        for k in ref:
            assert np.array_equal(m[k], ref[k]), (p["nx"], n, k)


def _kernels(run, sync):
    import torch
    from torch.profiler import ProfilerActivity, profile
    run()
    sync()
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            run()
            sync()
        torch.cuda.synchronize()
        names = [e.name for e in prof.events() if "lbmx::" in e.name and "advance" not in e.name]
    if not names:
        pytest.skip("no kernel trace on this machine")
    return [n.split("lbmx::")[1].split("<")[0].split("_kernel")[0] for n in names]


# (grid, form, steps, kernels): the measured figures stand at default_plan
LAST = [((1030, 515), "fp32", 1, ["pair"]), ((1030, 515), "fp32", 2, ["pair"]),
        ((1030, 515), "fp32", 3, ["march"]), ((1030, 515), "fp32", 6, ["march", "pair"]),
        ((1030, 515), "fp16", 3, ["step"] * 3), ((1030, 515), "fp16", 5, ["march", "step"]),
        ((2620, 1000), "fp32", 7, ["march", "pair"]), ((2620, 1000), "fp32", 4, ["march"]),
        ((3310, 1600), "fp16", 7, ["march", "march"]), ((3310, 1600), "fp16", 2, ["step"] * 2),
        ((3310, 1600), "fp16sr", 3, ["step"] * 3), ((128, 32), "fp32", 1, ["step"]),
        ((128, 32), "fp16", 9, ["stack", "step"]), ((128, 32), "fp32", 2, ["stack"]),
        ((800, 210), "fp32", 2, ["pair"])]


@pytest.mark.parametrize("grid,precision,steps,kernels", LAST, ids=str)
def test_kernels_of_the_last_steps(grid, precision, steps, kernels):
    from paper_1002_3028_amd import lbm
    p, inlet = _jet(*grid)
    with lbm.Solver(p, precision) as s:
        s.set_inlet(*inlet)
        assert _kernels(lambda: s.step(steps), s.sync) == kernels
    need = lbm.bytes_required(p, precision)
    with lbm.Batch(need + (1 << 20), 1, precision) as b:
        b.admit(p, inlet, 1 << 40)
        assert _kernels(lambda: b.run(steps), b.sync) == kernels

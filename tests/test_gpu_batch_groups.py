"""How a batch's jets are shared out over cohorts, seen by the kernel launches
of a group (torch's profiler): it follows the number of streams, also when that
changes between runs, and never changes a result."""
import collections
import warnings

import numpy as np
import pytest

from gpu_common import noisy_inlet, require_gpu, tiny_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _launches(b, k):
    """Graph launches and step kernels of one run of k steps."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    b.run(k)  # (captures)
    b.sync()
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            b.run(k)
            b.sync()
        torch.cuda.synchronize()
        seen = collections.Counter(e.name for e in prof.events())
    graphs = sum(n for name, n in seen.items() if "GraphLaunch" in name)
    steps = sum(n for name, n in seen.items() if "lbmx::" in name and "advance" not in name)
    if not steps:
        pytest.skip("no kernel trace on this machine")
    return graphs, steps


def _uneven():
    sizes = [(512, 128), (300, 70), (1500, 200), (700, 150), (512, 140), (640, 160)]
    return [(tiny_params(nx, nr, "jet", q % 2), noisy_inlet(nr, 3, q)) for q, (nx, nr)
            in enumerate(sizes)]


def test_cohorts_follow_the_number_of_streams():
    """Six FP16 jets (40 MB of buffers) share two streams evenly and run as one
    cohort on one stream, whichever came first; the fields are those of the
    jets run alone."""
    from paper_1002_3028_amd import lbm
    jets = _uneven()
    taken = 0
    with lbm.Batch(1 << 28, 8, "fp16") as b:
        slots = [b.admit(p, inlet, 1 << 40) for p, inlet in jets]
        for n in (1, 2, 1, 3, 2):
            b.set_streams(n)
            graphs, steps = _launches(b, 20)
            taken += 40
            assert graphs == n, (n, graphs, steps)
        got = [b.moments(s) for s in slots]
    for (p, inlet), m in zip(jets, got):
        with lbm.Solver(p, "fp16", tile_shape=0) as s:
            if inlet is not None:
                s.set_inlet(*inlet)
            s.step(taken)
            ref = s.moments()
        for key in ref:
            assert np.array_equal(m[key], ref[key]), (p["nx"], key)


def test_short_groups_run_as_one_cohort():
    """Jets that one cohort holds are split over two streams only for groups
    worth it, from the second run in a row on."""
    from paper_1002_3028_amd import lbm
    with lbm.Batch(1 << 28, 8, "fp16") as b:
        for p, inlet in _uneven():
            b.admit(p, inlet, 1 << 40)
        assert _launches(b, 2)[0] == 1
        assert _launches(b, 20)[0] == 2  # (two runs of 20)
        b.run(2)
        b.run(20)
        assert _launches(b, 20)[0] == 2
        b.run(2)
        assert _launches(b, 2)[0] == 1


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp16sr"])
def test_regrouped_jets_keep_their_bits(precision):
    """Runs of lengths that change how the jets are shared out, while one after
    another stops: each jet equals itself alone with one step per launch."""
    from paper_1002_3028_amd import lbm
    jets = [(p, inlet, 40 + 61 * q) for q, (p, inlet) in enumerate(_uneven())]
    with lbm.Batch(1 << 28, 8, precision) as b:
        slots = [b.admit(*j) for j in jets]
        for k in (1, 2, 60, 60, 3, 2, 1, 70, 70, 70, 5, 5, 1, 1):
            b.run(k)
        assert [b.poll(s) for s in slots] == [n for _, _, n in jets]
        got = [b.moments(s) for s in slots]
    for (p, inlet, n), m in zip(jets, got):
        with lbm.Solver(p, precision, tile_shape=0) as s:
            s.set_inlet(*inlet)
            s.step(n)
            ref = s.moments()
        for key in ref:
            assert np.array_equal(m[key], ref[key]), (p["nx"], n, key)


def test_more_group_lengths_than_graphs_are_kept():
    """Groups of 300 lengths, each captured when it first comes, more than the
    batch keeps, on two streams: the jets equal themselves run alone."""
    from paper_1002_3028_amd import lbm
    lengths = list(range(1, 301)) + [1, 2, 299]
    jets = [(tiny_params(64, 20, "jet", 1), noisy_inlet(20, 3, 1), 1 << 40),
            (tiny_params(59, 30, "jet", 0), noisy_inlet(30, 4, 2), 20000)]
    with lbm.Batch(1 << 26, 2, "fp16") as b:
        b.set_cohort_bytes(1)  # (a cohort each)
        slots = [b.admit(*j) for j in jets]
        for k in lengths:
            b.run(k)
        steps = [b.poll(s) for s in slots]
        assert steps == [sum(lengths), 20000]
        got = [b.moments(s) for s in slots]
    for (p, inlet, _), n, m in zip(jets, steps, got):
        with lbm.Solver(p, "fp16", tile_shape=0, graph_steps=50) as s:
            s.set_inlet(*inlet)
            s.step(n)
            ref = s.moments()
        for key in ref:
            assert np.array_equal(m[key], ref[key]), (p["nx"], key)

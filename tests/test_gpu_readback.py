"""Fields and populations out and in, at the sizes where the path changes:
results of up to 1 MiB come through pinned memory, larger ones in pieces of
64 MiB (rows of the fields, planes of the populations)."""
import numpy as np
import pytest

from gpu_common import host_threads, rel_err, require_gpu, tiny_params

pytestmark = pytest.mark.gpu

# (nx, nr): populations of exactly 1 MiB or less and just more (10 082 nodes),
# fields of exactly 1 MiB and just more (32 768 nodes), planes in several
# pieces, rows in several pieces
GRIDS = [(2, 2), (71, 142), (71, 143), (256, 128), (257, 128), (1100, 620), (2100, 1010)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("nx,nr", GRIDS)
def test_round_trip_and_fields(nx, nr):
    """Populations read back are those set (they are exact in FP32), the
    moments agree with the oracle's of the same populations to 2e-6 (FP32 sums
    of nine populations), and a value that is not finite anywhere leaves the
    state as it was."""
    import oracle
    from paper_1002_3028_amd import lbm
    p = tiny_params(nx, nr, "closed", 1)
    rng = np.random.default_rng(nx * nr)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]
    f = (w * rng.uniform(0.95, 1.05, (9, nr, nx))).astype(np.float32).astype(np.float64)
    g = rng.uniform(0.1, 0.2, (4, nr, nx)).astype(np.float32).astype(np.float64)
    with lbm.Solver(p, "fp32") as s, oracle.RefSolver(p, threads=host_threads()) as r:
        s.set_populations(f, g, 3)
        r.set_populations(f, g, 3)
        m, mr = s.moments(), r.moments()
        for bad_f, bad_g in ((None, (3, nr - 1, nx - 1)), ((0, 0, 0), None)):
            f2, g2 = f + 0.01, g.copy()
            if bad_g:
                g2[bad_g] = np.inf
            if bad_f:
                f2[bad_f] = np.nan
            with pytest.raises(lbm.LbmError) as e:
                s.set_populations(f2, g2, 8)
            assert e.value.code == lbm.EINVAL and s.step_count == 3
        f1, g1 = s.get_populations()
    assert np.array_equal(f1, f) and np.array_equal(g1, g)
    scale = np.abs(np.hypot(mr["ux"], mr["ur"])).max()
    assert rel_err(m["rho"], mr["rho"]) < 2e-6 and rel_err(m["T"], mr["T"]) < 2e-6
    assert np.abs(m["ux"] - mr["ux"]).max() < 2e-6 * max(scale, 1)
    assert np.abs(m["ur"] - mr["ur"]).max() < 2e-6 * max(scale, 1)


def test_batch_profiles_while_others_run():
    """Profiles of running and finished jets, with and without work queued
    since the last extraction, equal the moments' edges taken after a sync."""
    from paper_1002_3028_amd import lbm
    jets = [(tiny_params(300, 90, "jet", 1), 1 << 40), (tiny_params(64, 20, "jet", 0), 25)]
    with lbm.Batch(1 << 28, 4, "fp32") as b, lbm.Batch(1 << 28, 4, "fp32") as c:
        sb, sc = ([x.admit(p, None, n) for p, n in jets] for x in (b, c))
        for k in (10, 10, 10, 7):
            b.run(k)
            c.run(k)
            c.sync()
            for q, w in zip(sb, sc):
                for _ in range(2):
                    pr, m = b.profiles(q), c.moments(w)
                    assert np.array_equal(pr["ux_axis"], m["ux"][0])
                    assert np.array_equal(pr["T_axis"], m["T"][0])
                    assert np.array_equal(pr["ux_exit"], m["ux"][:, -1])
                    assert np.array_equal(pr["T_exit"], m["T"][:, -1])


@pytest.mark.parametrize("nx,nr", [(3000000, 2), (4200, 4100)])
def test_pieces_stay_small(nx, nr):
    """A row of fields (96 MB) or a plane of populations (138 MB) larger than a
    piece: reading fields and populations back takes at most 64 MiB of device
    memory (allocations are in steps of 2 MiB), restoring them 52 bytes a node
    more, and the values are those of the profiles and the ones set."""
    import torch
    from paper_1002_3028_amd import lbm
    p = tiny_params(nx, nr, "closed", 1)
    rng = np.random.default_rng(nx)
    line = rng.uniform(0.95, 1.05, nx + 12).astype(np.float32).astype(np.float64)

    def values(k):
        return np.stack([(0.1 + 0.01 * q) * np.broadcast_to(line[q:q + nx], (nr, nx)) *
                         (1.0 + np.arange(nr) % 3)[:, None] for q in range(k)]
                        ).astype(np.float32).astype(np.float64)
    f, g = values(9), values(4)
    piece, slack = 64 << 20, 4 << 20

    def used():
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free

    with lbm.Solver(p, "fp32") as s:
        s.sync()
        u0 = used()
        m = s.moments()
        s.get_populations()
        u1 = used()
        s.set_populations(f, g, 3)
        u2 = used()
        print(f"{nx}x{nr}: reading {u1 - u0}, restoring {u2 - u1}", flush=True)
        assert u1 - u0 <= piece + slack
        assert u2 - u0 <= 52 * nx * nr + piece + slack
        f1, g1 = s.get_populations()
        assert np.array_equal(f1, f) and np.array_equal(g1, g)
        m, pr = s.moments(), s.profiles()
        assert np.array_equal(pr["ux_axis"], m["ux"][0])
        assert np.array_equal(pr["T_axis"], m["T"][0])
        assert np.array_equal(pr["ux_exit"], m["ux"][:, -1])
        assert np.array_equal(pr["T_exit"], m["T"][:, -1])
    with lbm.Batch(lbm.bytes_required(p) + (1 << 20), 1, "fp32") as b:
        slot = b.admit(p, None, 10)
        b.run(4)
        u0 = used()
        m = b.moments(slot)
        assert used() - u0 <= piece + slack
        pr = b.profiles(slot)
        assert np.array_equal(pr["ux_axis"], m["ux"][0])
        assert np.array_equal(pr["T_exit"], m["T"][:, -1])


def test_batch_fields_do_not_wait_for_other_streams():
    """Large fields of a batch's jet come back while work that the program put
    on the default stream (about 150 ms) is still running.  (Streams are spread
    over a few hardware queues, and those on one queue run in order, so one of
    four batches, whose streams land on different queues, has to show it.)"""
    import contextlib

    import torch
    from paper_1002_3028_amd import lbm
    p = tiny_params(1100, 620, "jet", 1)
    a = torch.ones(8192, 8192, device="cuda", dtype=torch.bfloat16)
    a @ a
    torch.cuda.synchronize()
    waited = []
    with contextlib.ExitStack() as stack:
        while len(waited) < 4 and all(waited):
            b = stack.enter_context(lbm.Batch(1 << 28, 1, "fp32"))
            slot = b.admit(p, None, 10)
            b.run(10)
            b.sync()
            ref = b.moments(slot)
            other = torch.cuda.Event()
            for _ in range(200):
                a @ a
            other.record()
            m = b.moments(slot)
            waited.append(other.query())
            torch.cuda.synchronize()
            for k in ref:
                assert np.array_equal(m[k], ref[k]), k
    assert not all(waited)


@pytest.mark.parametrize("nx,nr", [(4000, 96), (4001, 96), (2, 5000), (70000, 3)])
def test_profiles_of_long_grids(nx, nr):
    """Profiles of 64 KiB and just more (whose memory comes when they are asked
    for), and of more than the fields' direct path takes, equal the moments'
    edges, before and after fields and populations have used the same memory."""
    from paper_1002_3028_amd import inputs, lbm
    p = tiny_params(nx, nr, "closed", 1)
    with lbm.Solver(p, "fp32") as s:
        s.set_state(*inputs.perturbed_state(nx, nr, seed=nx, noise=0.3))
        for n in (0, 3, 4):
            s.step(n)
            pr, m = s.profiles(), s.moments()
            again = s.profiles()
            s.get_populations()
            for k, ref in (("ux_axis", m["ux"][0]), ("T_axis", m["T"][0]),
                           ("ux_exit", m["ux"][:, -1]), ("T_exit", m["T"][:, -1])):
                assert np.array_equal(pr[k], ref) and np.array_equal(again[k], ref), (n, k)

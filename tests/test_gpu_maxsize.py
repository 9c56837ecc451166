"""The largest grid the library accepts: 8247 x 4961 nodes, whose 13 FP32
planes (pitch 8320, 4963 rows with the ghost ring) take 2 147 192 320 bytes,
just under the 2^31 reach of the kernels' 32-bit byte offsets (one more
column or row is refused, `test_abi_cpu.py`).  Both sizes are ragged against
the tiles.  The state is rough at node level (every node differs from its
neighbours by about a third of the field's amplitude), so a wrong offset
anywhere in the buffer shows as an O(1) error against the FP64 oracle:

* FP32, two steps per launch in graphs of 50 steps (the benchmark's launch),
  within 1e-4 of the field scale on u and T after 3 steps (a pair and a single
  step), and bit-identical to the one-step kernel and to the single-buffer
  layout; profiles within 1e-4 and the FP64 mass and energy sums within 1e-6;
* FP16 storage within 5e-3 of the scale: the check is on addressing, and
  binary16 rounding of the stored deviations (half an ulp is 2.4e-4 of a
  value) over three steps stays well below it.
"""
import json

import numpy as np
import pytest

from gpu_common import host_threads, rel_err, require_gpu, speed

pytestmark = pytest.mark.gpu

NX, NR, STEPS = 8247, 4961, 3


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.fixture(scope="module")
def case():
    import oracle
    from paper_1002_3028_amd import inputs
    p, inlet, _ = inputs.workload_large(NX, NR, n_t=STEPS + 1)
    st = inputs.perturbed_state(NX, NR, seed=8247, amp=0.02, T_mean=0.5, T_amp=0.2, noise=0.5)
    print(f"max grid {NX}x{NR}: oracle, {STEPS} steps", flush=True)
    with oracle.RefSolver(p, threads=host_threads()) as r:
        r.set_state(*st)
        r.set_inlet(*inlet)
        r.step(STEPS)
        ref = (r.moments(), r.profiles(), r.conservation())
    return p, inlet, st, ref


def _run(p, inlet, st, precision, **kw):
    from paper_1002_3028_amd import lbm
    print(f"max grid {NX}x{NR}: {precision} {kw}", flush=True)
    with lbm.Solver(p, precision, **kw) as s:
        s.set_state(*st)
        s.set_inlet(*inlet)
        s.step(STEPS)
        return s.moments(), s.profiles(), s.conservation()


def _errors(got, ref):
    m, pr, cons = got
    mr, prr, consr = ref
    return {"u": rel_err(speed(m), speed(mr)), "T": rel_err(m["T"], mr["T"]),
            "rho-1": rel_err(m["rho"] - 1.0, mr["rho"] - 1.0),
            "profiles": max(rel_err(pr[k], prr[k]) for k in pr),
            "mass": abs(cons[0] - consr[0]) / abs(consr[0]),
            "energy": abs(cons[1] - consr[1]) / abs(consr[1])}


def test_fp32_largest_grid(case):
    from paper_1002_3028_amd import lbm
    p, inlet, st, ref = case
    pair = _run(p, inlet, st, "fp32", graph_steps=50)
    e = _errors(pair, ref)
    print(json.dumps({"grid": f"{NX}x{NR}", "precision": "fp32", **e}))
    assert e["u"] < 1e-4 and e["T"] < 1e-4 and e["profiles"] < 1e-4
    assert e["mass"] < 1e-6 and e["energy"] < 1e-6
    one_step = [q for q, i in enumerate(lbm.tile_shape_infos()) if i["steps"] == 1][0]
    for kw in ({"tile_shape": one_step}, {"layout": "single"}):
        other = _run(p, inlet, st, "fp32", **kw)
        for key in pair[0]:
            assert np.array_equal(other[0][key], pair[0][key]), (kw, key)
        assert other[2] == pair[2], kw
        del other


def test_fp16_largest_grid(case):
    p, inlet, st, ref = case
    e = _errors(_run(p, inlet, st, "fp16"), ref)
    print(json.dumps({"grid": f"{NX}x{NR}", "precision": "fp16", **e}))
    assert e["u"] < 5e-3 and e["T"] < 5e-3 and e["profiles"] < 5e-3


@pytest.mark.parametrize("precision", ["fp32", "fp16", "fp16sr"])
def test_default_shape_largest_grid_full_launches(case, precision):
    """Thirteen steps in the shape a solver takes by itself (marching): launches
    with all their levels, which three steps do not reach, and one of the rest;
    bit-identical to one step per launch."""
    from paper_1002_3028_amd import lbm
    p, inlet, st, _ = case
    got = []
    for kw in ({}, {"tile_shape": 0}):
        print(f"max grid {NX}x{NR}: {precision} {kw}", flush=True)
        with lbm.Solver(p, precision, **kw) as s:
            s.set_state(*st)
            s.set_inlet(*inlet)
            s.step(13)
            got.append((s.moments(), s.conservation()))
    for key in got[0][0]:
        assert np.array_equal(got[0][0][key], got[1][0][key]), key
    assert got[0][1] == got[1][1]

"""The bench's roofline names the bound of the kernel that ran: HBM by the
algorithmic bytes with one step per launch; with several, whose rate by those
bytes is no bandwidth, vector-ALU issue or HBM by the bytes moved, and no
fraction of a peak above one."""
import pytest

NODES = 2048 * 512


def _shape(steps, by=4):
    return {"steps": steps, "by": by}


@pytest.fixture
def bench(monkeypatch):
    import bench
    monkeypatch.setattr(bench, "read_traffic", lambda name: 150.6e6)
    monkeypatch.setattr(bench, "read_summary", lambda name, key: 266.3)
    monkeypatch.setattr(bench, "read_trace_us", lambda name, kernel: None)
    return bench


def test_one_step_is_bound_by_algorithmic_bytes(bench):
    r = bench.roofline_block("fp32", _shape(1), NODES, 17.5e-3, "t", tag="2048x512")
    assert r["bound"] == "hbm" and r["unit"] == "GB/s" and r["peak"] == 8000.0
    assert r["achieved"] == r["effective_GBps"] == pytest.approx(104 * NODES / 17.5e-6 / 1e9, rel=1e-3)
    assert r["frac"] == pytest.approx(r["achieved"] / 8000.0, rel=1e-3)


def test_four_steps_are_bound_by_issue(bench):
    r = bench.roofline_block("fp32", _shape(4), NODES, 9.69e-3, "t", tag="2048x512")
    assert r["bound"] == "valu" and r["unit"] == "T lane-op/s"
    assert r["frac"] == r["alu"]["frac"] == pytest.approx(266.3 * NODES / 9.69e-6 / 39.32e12, rel=1e-2)
    assert r["effective_GBps"] > 8000.0 and r["frac"] < 1.0
    assert r["traffic_GBps"] == pytest.approx(150.6e6 / (4 * 9.69e-6) / 1e9, rel=1e-3)


def test_without_counters_the_bytes_each_launch_must_move(bench, monkeypatch):
    monkeypatch.setattr(bench, "read_traffic", lambda name: None)
    monkeypatch.setattr(bench, "read_summary", lambda name, key: None)
    for tag in (None, "2048x512"):
        r = bench.roofline_block("fp32", _shape(4), NODES, 9.69e-3, "t", tag=tag)
        assert r["bound"] == "hbm" and r["frac"] < 1.0
        assert r["achieved"] == pytest.approx(104 * NODES / (4 * 9.69e-6) / 1e9, rel=1e-3)

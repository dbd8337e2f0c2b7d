"""Grid engine, windowed forms (one wavefront per workgroup, and several):
parity with the CPU oracle where they can go wrong -- many workgroups and few,
several nodes and sides per workgroup, buffers of one line (every head refused
until its credit is back), batches of more entries than one read takes, windows
shorter and longer than a buffer's drain, both arbitrations, deadlocks, the
cycle guard at its last cycle.  Which form a load takes by itself is checked in
tests/test_host_plans.py."""
from __future__ import annotations

import numpy as np
import pytest

import sim_inputs as si
from tests.test_gpu_parity import check_engine, simmod, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def tree(k, lines, cap, lo, hi, arb, seed):
    rng = np.random.default_rng(seed)
    w = si.fat_tree(k, lat_seed=seed, lat_lo=lo, lat_hi=hi, cap=cap, nbytes=128 * lines, arb=arb)
    w.credit = rng.integers(np.maximum(2, w.lat - lo // 2), w.lat + lo // 2 + 2).astype(np.int32)
    return w


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("k,lines,cap,lo,hi", [(4, 6, 1, 32, 40), (4, 40, 100, 64, 90), (6, 3, 7, 40, 70), (8, 2, 32, 100, 300),
                                               (4, 5, 3, 2, 6)])
def test_fat_tree(simmod, oracle_lib, k, lines, cap, lo, hi, arb):
    assert check_engine(simmod, oracle_lib, tree(k, lines, cap, lo, hi, arb, 70 + k), "grid", must_run=True) == 1


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("wgs", [1, 2, 7, 33])
def test_workgroups(simmod, oracle_lib, wgs, arb, monkeypatch):
    """From every node in one workgroup (more sides than lanes: the
    multi-wave form) to one node each."""
    monkeypatch.setenv("SIMGPU_GRID_WGS", str(wgs))
    assert check_engine(simmod, oracle_lib, tree(4, 8, 9, 33, 50, arb, 5), "grid", must_run=True) == 1


@pytest.mark.parametrize("cap", [2, 4, 40])
def test_deadlock_or_end(simmod, oracle_lib, cap):
    """All-to-all on a torus: shallow buffers deadlock, deep ones end."""
    w = si.torus2d(4, 4, n_scenarios=1, seed=3, bws=(1, 1), lat_lo=34, lat_hi=40, depths=(cap,), nbytes=128 * 24,
                   coll=si.COLL_ALLTOALL, arb=1)
    w.credit = (w.lat + 3).astype(np.int32)
    check_engine(simmod, oracle_lib, w, "grid", must_run=True)


def test_max_cycles(simmod, monkeypatch):
    monkeypatch.setenv("SIMGPU_ENGINE", "grid")
    s = simmod.Simulator.from_workload(tree(4, 5, 6, 32, 60, 1, 9))
    mk = int(s.run().makespan[0])
    assert s.run(max_cycles=mk - 2).status == simmod.SIM_ERR_MAX_CYCLES
    r = s.run(max_cycles=mk - 1)  # the last cycle that moves a line
    assert r.status == simmod.SIM_OK and int(r.makespan[0]) == mk
    s.close()


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("wgs", [2, 8])
def test_max_cycles_many_sides(simmod, oracle_lib, wgs, arb, monkeypatch):
    """More sides per workgroup than lanes (the multi-wave form, over several
    workgroups): a run that ends at the guard's last cycle has ended."""
    monkeypatch.setenv("SIMGPU_ENGINE", "grid")
    monkeypatch.setenv("SIMGPU_GRID_WGS", str(wgs))
    w = tree(8, 2, 6, 5, 9, arb, 9)
    want = oracle_lib.simulate_workload(w)
    s = simmod.Simulator.from_workload(w)
    assert s.run(max_cycles=want.makespan - 2).status == simmod.SIM_ERR_MAX_CYCLES
    for mc in (want.makespan - 1, want.makespan, 0):  # the last cycle that moves a line is makespan - 1
        r = s.run(max_cycles=mc)
        assert r.status == simmod.SIM_OK and int(r.makespan[0]) == want.makespan
        assert np.array_equal(r.completion[0].cpu().numpy().view(np.uint32), want.completion)
        assert np.array_equal(r.tx_lines[0].cpu().numpy().astype(np.uint64), want.tx_lines)
    s.close()


# The multi-wave form, which short windows with many sides per workgroup take,
# over two and more workgroups.

def multi(monkeypatch, wgs=None):
    monkeypatch.setenv("SIMGPU_GRID_WINDOW", "multi")
    if wgs:
        monkeypatch.setenv("SIMGPU_GRID_WGS", str(wgs))


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("k,lines,cap,lo,hi", [(4, 6, 1, 32, 40), (4, 40, 100, 64, 90), (6, 3, 7, 2, 5), (8, 2, 32, 3, 7),
                                               (4, 5, 3, 2, 6)])
def test_fat_tree_multi(simmod, oracle_lib, k, lines, cap, lo, hi, arb, monkeypatch):
    multi(monkeypatch)
    assert check_engine(simmod, oracle_lib, tree(k, lines, cap, lo, hi, arb, 80 + k), "grid", must_run=True) == 1


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("wgs", [2, 7, 32])
def test_workgroups_multi(simmod, oracle_lib, wgs, arb, monkeypatch):
    multi(monkeypatch, wgs)
    assert check_engine(simmod, oracle_lib, tree(4, 8, 9, 6, 50, arb, 5), "grid", must_run=True) == 1


@pytest.mark.parametrize("cap", [2, 4, 40])
def test_deadlock_or_end_multi(simmod, oracle_lib, cap, monkeypatch):
    multi(monkeypatch, 7)
    w = si.torus2d(4, 4, n_scenarios=1, seed=3, bws=(1, 1), lat_lo=5, lat_hi=9, depths=(cap,), nbytes=128 * 24,
                   coll=si.COLL_ALLTOALL, arb=1)
    w.credit = (w.lat + 3).astype(np.int32)
    check_engine(simmod, oracle_lib, w, "grid", must_run=True)


def test_max_cycles_multi(simmod, monkeypatch):
    multi(monkeypatch, 8)
    test_max_cycles(simmod, monkeypatch)


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("lo", [2, 3, 4, 6, 8])
def test_short_windows(simmod, oracle_lib, lo, arb):
    """The form that the load takes by itself, on both sides of the rule."""
    for k in (4, 8):
        assert check_engine(simmod, oracle_lib, tree(k, 2, 5, lo, lo + 3, arb, 90 + lo), "grid", must_run=True) == 1

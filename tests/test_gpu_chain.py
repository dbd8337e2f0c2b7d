"""Wave engine, chain loops (lined-up graphs with one flow on and one out per
link): parity with the CPU oracle where they can go wrong -- buffers of one to
three lines, several scenarios of a wave that idle, end and deadlock at
different cycles, ranges of one line, two and more predecessors per range,
more than eight, per-chunk dependencies, both arbitrations, the cycle guard at
its last cycle, stopped scenarios next to running ones -- and against the
loops they replace; then the general round-robin loops at eight lines, which are
compiled apart.  Which loop a load takes is checked in tests/test_host_plans.py."""
from __future__ import annotations

import numpy as np
import pytest

import sim_inputs as si
from tests.test_gpu_parity import check_engine, simmod, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
@pytest.mark.parametrize("coll", [si.COLL_RING_ALLREDUCE, si.COLL_RING_ALLGATHER])
@pytest.mark.parametrize("bws,c", [((1,), 1), ((1,), 7), ((2,), 5), ((1, 2, 4), 6), ((4, 8), 9), ((3,), 4)])
def test_torus_ring(simmod, oracle_lib, arb, dep, coll, bws, c):
    w = si.torus2d(4, 4, n_scenarios=14, seed=31 + arb + len(bws) + c, bws=bws, lat_lo=1, lat_hi=25,
                   depths=(1, 2, 3, 5, 16, 33), nbytes=128 * 16 * c, arb=arb, coll=coll)
    w.dep = dep
    check_engine(simmod, oracle_lib, w, "wave", must_run=True)


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
@pytest.mark.parametrize("p,b,coll", [(3, 1, si.COLL_DIRECT_ALLREDUCE), (4, 1, si.COLL_DIRECT_ALLREDUCE),
                                      (8, 2, si.COLL_DIRECT_ALLREDUCE), (8, 4, si.COLL_RHD_ALLREDUCE),
                                      (8, 1, si.COLL_RHD_ALLREDUCE), (7, 1, si.COLL_DBT_ALLREDUCE),
                                      (6, 3, si.COLL_DBT_ALLREDUCE), (5, 2, si.COLL_RING_ALLREDUCE)])
def test_mesh(simmod, oracle_lib, arb, dep, p, b, coll):
    w = si.full_mesh(p, b=b, L=6, cap=4, coll=coll, nbytes=128 * 6 * p, arb=arb)
    w.lat = np.random.default_rng(p).integers(1, 12, w.n_links).astype(np.int32)
    w.dep = dep
    assert check_engine(simmod, oracle_lib, w, "wave", must_run=True) == 1


@pytest.mark.parametrize("b", [1, 2, 4])
@pytest.mark.parametrize("n_preds", [2, 3, 9, 12])
def test_predecessors(simmod, oracle_lib, n_preds, b):
    """Single-line ranges, each waiting on up to n_preds flows of a mesh."""
    rng = np.random.default_rng(600 + n_preds)
    p, n = 5, 220
    src = rng.integers(0, p, n).astype(np.int32)
    dst = ((src + rng.integers(1, p, n)) % p).astype(np.int32)
    pptr, pidx = [0], []
    for x in range(n):
        k = min(x, int(rng.integers(0, n_preds + 1)))
        pidx += sorted(int(v) for v in rng.choice(x, size=k, replace=False)) if k else []
        pptr.append(len(pidx))
    w = si.full_mesh(p, b=b, L=3, cap=3, nbytes=128)
    check_engine(simmod, oracle_lib, w, "wave", txns=(src, dst, np.array(pptr, np.int64), np.array(pidx, np.int64)),
                 must_run=True)


@pytest.mark.parametrize("bws", [(1,), (2,), (4,)])
def test_max_cycles(simmod, bws, monkeypatch):
    monkeypatch.setenv("SIMGPU_ENGINE", "wave")
    w = si.torus2d(4, 4, n_scenarios=3, seed=2, bws=bws, lat_lo=9, lat_hi=9, depths=(6,), nbytes=128 * 16 * 4)
    s = simmod.Simulator.from_workload(w)
    r = s.run()
    mk, cyc = int(r.makespan[0]), r.cycles.copy()
    assert s.run(max_cycles=mk - 2).status == simmod.SIM_ERR_MAX_CYCLES
    r = s.run(max_cycles=mk - 1)  # the last cycle that moves a line
    assert r.status == simmod.SIM_OK and int(r.makespan[0]) == mk and np.array_equal(r.cycles, cyc)
    s.close()


@pytest.mark.parametrize("arb,coll", [(0, si.COLL_RING_ALLREDUCE), (1, si.COLL_RING_ALLREDUCE),
                                      (0, si.COLL_RHD_ALLREDUCE)])
@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
@pytest.mark.parametrize("bws", [(1,), (2,), (4,), (8,)])
def test_stopped_by_guard(simmod, oracle_lib, bws, dep, arb, coll, monkeypatch):
    """Scenarios of one wave that the cycle guard stops early, late and not at
    all: each leaves exactly what the oracle leaves when stopped at the same
    cycle, whatever the wave's other scenarios still do."""
    monkeypatch.setenv("SIMGPU_ENGINE", "wave")
    w = si.torus2d(4, 2, n_scenarios=12, seed=51, bws=bws, lat_lo=2, lat_hi=40, depths=(2, 5, 16), nbytes=128 * 8 * 24,
                   arb=arb, coll=coll)
    w.dep = dep
    if coll == si.COLL_RHD_ALLREDUCE:
        w.order = si.gray_torus_order(4, 2)
    s = simmod.Simulator.from_workload(w)
    mks = np.sort([oracle_lib.simulate_workload(w, k).makespan for k in range(w.n_scenarios)])
    for mc in (1, int(mks[0]) // 2, int(mks[0]) + 3, int(mks[len(mks) // 2]), int(mks[-1]) - 2):
        outs = s.alloc_outputs()
        for o in outs:
            o.fill_(-1)
        r = s.run(max_cycles=mc, outs=outs)
        for k in range(w.n_scenarios):
            want = oracle_lib.simulate_workload(w, k, max_cycles=mc)
            assert int(r.scenario_status[k]) == {"OK": 0, "MAX_CYCLES": 8}[want.status_name], (mc, k)
            assert np.array_equal(r.tx_lines[k].cpu().numpy().astype(np.uint64), want.tx_lines), (mc, k)
            assert np.array_equal(r.busy_cycles[k].cpu().numpy().astype(np.uint64), want.busy_cycles), (mc, k)
            # (lines that did not complete keep the buffer's fill)
            assert np.array_equal(r.completion[k].cpu().numpy().view(np.uint32), want.completion), (mc, k)
    s.close()


@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
def test_same_as_shift_loop(simmod, oracle_lib, dep, monkeypatch):
    """The same bytes and processed cycles as the shift loop."""
    w = si.torus2d(4, 4, n_scenarios=40, seed=8, bws=(1, 2, 4), lat_lo=3, lat_hi=60, depths=(4, 16, 40),
                   nbytes=128 * 16 * 40)
    w.dep = dep
    got = []
    for loop in ("shift", ""):
        monkeypatch.setenv("SIMGPU_WAVE_LOOP", loop)
        s = simmod.Simulator.from_workload(w)
        r = s.run()
        assert r.status == simmod.SIM_OK
        got.append([a.cpu().numpy() for a in (r.completion, r.tx_lines, r.busy_cycles, r.makespan)] + [r.cycles])
        s.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))
    assert got[0][4][0] == oracle_lib.simulate_workload(w, 0).processed_cycles


EIGHT_LINES = [(4, 2, si.COLL_DBT_ALLREDUCE), (4, 4, si.COLL_RHD_ALLREDUCE), (3, 2, si.COLL_DIRECT_ALLREDUCE)]


@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
@pytest.mark.parametrize("bws", [(8,), (5, 8), (1, 2, 4, 8)])
def test_general_round_robin_eight_lines(simmod, oracle_lib, bws, dep):
    """The round-robin loops of graphs that are not lined up, at up to eight
    lines per cycle: several feeders per link (trees), several predecessors per
    range (halving-doubling, direct)."""
    for X, Y, coll in EIGHT_LINES:
        w = si.torus2d(X, Y, n_scenarios=9, seed=61, bws=bws, lat_lo=1, lat_hi=12, depths=(9, 24, 40),
                       nbytes=128 * X * Y * 14, arb=1, coll=coll)
        w.dep = dep
        check_engine(simmod, oracle_lib, w, "wave", must_run=True)


@pytest.mark.parametrize("b,cap", [(8, 40), (6, 9), (8, 3)])
def test_general_round_robin_ring_of_links(simmod, oracle_lib, b, cap):
    """One feeder per link, on a cycle: the same loops with two request groups."""
    rp, ci = np.array([0, 1, 2, 3], np.int32), np.array([1, 2, 0], np.int32)
    rng = np.random.default_rng(b + cap)
    src = rng.integers(0, 3, 90).astype(np.int32)
    dst = ((src + rng.integers(1, 3, 90)) % 3).astype(np.int32)
    par = np.full(3, b, np.int32)
    w = si.Workload("ring3", 3, 3, rp, ci, 1, par, np.full(3, 2, np.int32), np.full(3, cap, np.int32), 1, -1, 0)
    check_engine(simmod, oracle_lib, w, "wave", txns=(src, dst, np.zeros(91, np.int64), np.zeros(0, np.int64)),
                 must_run=True)

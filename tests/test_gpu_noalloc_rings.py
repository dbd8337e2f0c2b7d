"""The allocation-free run of sweeps whose engine keeps its rings in device
memory: where those rings exceed the fixed scratch, the engine's LDS form runs
instead, with the bytes of sim_run (which has its own scratch)."""
from __future__ import annotations

import sys
from dataclasses import replace

import numpy as np
import pytest

import sim_inputs as si
from tests.test_zz_no_alloc import _run, simmod  # noqa: F401

pytestmark = pytest.mark.gpu


def workload(arb, bws, S):
    rng = np.random.default_rng(S + len(bws))
    w = si.fat_tree(4, lat_seed=S, lat_lo=2, lat_hi=12, nbytes=128 * 2, arb=arb)
    m = len(w.lat)
    return replace(w, n_scenarios=S, lat=np.tile(w.lat, S), bw=np.repeat(rng.choice(bws, S), m).astype(np.int32),
                   cap=np.repeat(rng.choice([5, 16], S), m).astype(np.int32))


# route (round-robin), lane (lowest id, several lines per cycle) and compact
# engine (lowest id, one line per cycle).  30 scenarios fit the scratch; the
# lane and compact engine's rings exceed it at 1100, where the route engine
# still has its rings in LDS: those are in device memory, and exceed the
# scratch, at 1700 (tests/test_host_plans.py checks the engines).
@pytest.mark.parametrize("arb,bws", [(si.ARB_ROUND_ROBIN, (1, 2, 4)), (si.ARB_LOWEST_ID, (1, 2)),
                                     (si.ARB_LOWEST_ID, (1,))])
@pytest.mark.parametrize("S", [30, 1100, 1700])
def test_noalloc_sweep(simmod, oracle_lib, arb, bws, S):  # noqa: F811
    w = workload(arb, bws, S)
    print(f"no-alloc sweep: arb={arb} bw={bws} S={S}", file=sys.stderr, flush=True)
    s = simmod.Simulator.from_workload(w)
    try:
        want = _run(simmod, s, False)
        got = _run(simmod, s, True)
    finally:
        s.close()
    assert want[0] == got[0] == 0
    assert np.array_equal(want[1], got[1]) and np.array_equal(want[2], got[2])
    for a, b in zip(want[3], got[3]):
        assert np.array_equal(a, b)
    for k in (0, S - 1):
        o = oracle_lib.simulate_workload(w, k)
        assert np.array_equal(got[3][0][k, :len(o.completion)].view(np.uint32), o.completion)


def test_noalloc_workgroup_in_place_of_route(simmod, oracle_lib):  # noqa: F811
    """Rings too deep for the scratch at the route engine's 16 B per entry: the
    workgroup engine's 12 B fit."""
    from tests.test_host_plans import deep_stars
    w, txns = deep_stars()
    s = simmod.Simulator.from_workload(w)
    try:
        s.load_transactions(*txns)
        want = _run(simmod, s, False)
        got = _run(simmod, s, True)
    finally:
        s.close()
    assert want[0] == got[0] == 0
    for a, b in zip(want[3], got[3]):
        assert np.array_equal(a, b)
    o = oracle_lib.simulate(w.n_nodes, w.n_endpoints, w.row_ptr, w.col_idx, w.bw, w.lat, w.cap, w.arb, txns=txns)
    assert np.array_equal(got[3][0][0].view(np.uint32), o.completion)
    assert np.array_equal(got[3][1][0].astype(np.uint64), o.tx_lines)

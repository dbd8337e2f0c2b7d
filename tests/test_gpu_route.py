"""Route engine (round-robin, one thread per traffic link, source-routed
lines): parity with the CPU oracle with its rings in LDS and in device
memory, at the edges of its forms -- one line per cycle and several, batches
of mixed bandwidths, one and several waves, rings of one entry, lines that
run over several ranges in a cycle, more predecessors than fit in registers,
per-chunk dependencies, idle jumps and deadlocks."""
from __future__ import annotations

import numpy as np
import pytest

import sim_inputs as si
from tests.test_gpu_parity import check_engine, run_engine, simmod, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

ENG = ["route", "routehbm"]


@pytest.mark.parametrize("engine", ENG)
@pytest.mark.parametrize("k,cap,lines", [(4, 1, 3), (4, 5, 12), (6, 3, 4), (8, 8, 2)])
def test_fat_tree(simmod, oracle_lib, engine, k, cap, lines):
    w = si.fat_tree(k, nbytes=128 * lines, cap=cap, lat_lo=1, lat_hi=9)
    assert check_engine(simmod, oracle_lib, w, engine, must_run=True) == 1


@pytest.mark.parametrize("engine", ENG)
@pytest.mark.parametrize("coll", [si.COLL_RING_ALLREDUCE, si.COLL_DBT_ALLREDUCE, si.COLL_DIRECT_ALLREDUCE])
@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
def test_fat_tree_dependencies(simmod, oracle_lib, engine, coll, dep):
    w = si.fat_tree(4, nbytes=128 * 16 * 3 * 2, cap=6, lat_lo=2, lat_hi=9, coll=coll)
    S, m = 5, w.n_links  # mixed bandwidths: every scenario runs its own loop
    w.n_scenarios = S
    w.lat = np.tile(w.lat, S)
    w.bw = np.repeat(np.array([1, 2, 3, 4, 1], np.int32), m)
    w.cap = np.repeat(np.array([6, 1, 9, 5, 2], np.int32), m)
    w.dep = dep
    check_engine(simmod, oracle_lib, w, engine, must_run=engine == "routehbm")


@pytest.mark.parametrize("engine", ENG)
@pytest.mark.parametrize("G,M,intra,fabric,lines", [(2, 3, (2, 4, 7), (1, 9, 8), 4), (8, 8, (2, 40, 64), (1, 200, 64), 1),
                                                    (3, 4, (4, 5, 3), (3, 7, 2), 5)])
def test_hierarchical(simmod, oracle_lib, engine, G, M, intra, fabric, lines):
    w = si.domains_leaf_spine(G, M, G, 2, intra=intra, fabric=fabric, nbytes=128 * G * M * lines)
    check_engine(simmod, oracle_lib, w, engine, must_run=engine == "routehbm")


@pytest.mark.parametrize("engine", ENG)
@pytest.mark.parametrize("p,b", [(12, 1), (12, 4), (10, 2)])
def test_many_predecessors(simmod, oracle_lib, engine, p, b):
    w = si.full_mesh(p, b=b, L=4, cap=5, coll=si.COLL_DIRECT_ALLREDUCE, nbytes=128 * 3 * p, arb=1)
    assert check_engine(simmod, oracle_lib, w, engine, must_run=True) == 1


@pytest.mark.parametrize("engine", ENG)
@pytest.mark.parametrize("seed", range(16))
def test_random_dags(simmod, oracle_lib, engine, seed):
    """Single-line ranges with random predecessors: range changes every
    line, offers over several ranges, void grants, deadlocks."""
    rng = np.random.default_rng(9100 + seed)
    n_end = int(rng.integers(2, 7))
    n, rp, ci, bw, lat, cap = si.random_graph(rng, n_end, int(rng.integers(0, 4)), int(rng.integers(0, 6)),
                                              bmax=int(rng.choice([1, 2, 3, 4])), Lmax=5, capmax=9, S=3)
    txns = si.random_dag(rng, n_end, int(rng.integers(1, 300)), max_preds=3)
    w = si.Workload("rand_route", n, n_end, rp, ci, 3, bw, lat, cap, 1, -1, 0)
    check_engine(simmod, oracle_lib, w, engine, txns=txns)


@pytest.mark.parametrize("engine", ENG)
def test_max_cycles(simmod, engine, monkeypatch):
    w = si.fat_tree(4, nbytes=128 * 4, cap=4, lat_lo=3, lat_hi=9)
    monkeypatch.setenv("SIMGPU_ENGINE", engine)
    s = simmod.Simulator.from_workload(w)
    mk = int(s.run().makespan[0])
    assert s.run(max_cycles=mk - 2).status == simmod.SIM_ERR_MAX_CYCLES
    r = s.run(max_cycles=mk - 1)  # the last cycle processed is makespan - 1
    assert r.status == simmod.SIM_OK and int(r.makespan[0]) == mk
    s.close()

"""The engine a load is given and the form it takes, on the CPU: the host
builder (api.cpp) built host-only against a stand-in HIP header whose device
memory is host memory, with a launcher that keeps what would have been
launched (tests/hip_host_stub)."""
from __future__ import annotations

import ctypes as C
import os
import shutil
import subprocess
from dataclasses import replace

import numpy as np
import pytest

import sim_inputs as si

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ENGINE = {"workgroup": 0, "lane": 1, "lanehbm": 2, "b1": 3, "wave": 4, "grid": 5, "resident": 6, "route": 7,
          "routehbm": 8}
NAME = {v: k for k, v in ENGINE.items()}

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def stub_path(tmp_path_factory):
    lib = tmp_path_factory.mktemp("plans") / "libsimgpu_plans.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", os.path.join(HERE, "hip_host_stub"), "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2606_10440_amd", "csrc", "api.cpp"),
                    os.path.join(HERE, "hip_host_stub", "engines_stub.cpp"), "-o", str(lib)], check=True)
    return str(lib)


@pytest.fixture
def plans(stub_path, monkeypatch):
    """The binding on the stand-in build."""
    from paper_2606_10440_amd import sim
    monkeypatch.setattr(sim, "LIB_PATH", stub_path)
    monkeypatch.setattr(sim, "_lib", None)
    monkeypatch.setenv("SIMGPU_STUB_DEVICE", "1")
    for v in ("SIMGPU_ENGINE", "SIMGPU_STUB_ALLOC_MAX", "SIMGPU_WAVE_LOOP", "SIMGPU_GRID_WGS", "SIMGPU_GRID_WINDOW"):
        monkeypatch.delenv(v, raising=False)
    L = sim.lib()
    L.stub_last.restype = C.c_int64
    L.stub_last.argtypes = [C.c_char_p]
    L.stub_blk_wave.restype = L.stub_wv_sc.restype = C.POINTER(C.c_int32)
    return sim


def last(sim, name):
    return int(sim.lib().stub_last(name.encode()))


def launch(sim, s, noalloc=False):
    """What a run of s launches: the engine's name."""
    (sim.sim_run_noalloc if noalloc else sim.sim_run)(s.ctx, 0, 1, 1, 1, 1, 0)  # (nothing is written)
    return NAME[last(sim, "engine")]


def sweep(w, S, bws, seed=1, cap=16):
    r = np.random.default_rng(seed)
    m = w.n_links
    return replace(w, n_scenarios=S, lat=np.tile(w.lat[:m], S), bw=np.repeat(r.choice(bws, S), m).astype(np.int32),
                   cap=np.full(S * m, cap, np.int32))


def deep_stars():
    """Four unconnected stars of 31 endpoints, 36 cables with deep buffers, all
    pairs of a star: round-robin, four lines per cycle, latencies beyond 16 bits."""
    p, stars = 31, 4  # endpoints around a switch; unconnected stars
    E = p * stars
    rp, ci = [0], []
    for u in range(E):
        ci.append(E + u // p)
        rp.append(len(ci))
    for q in range(stars):
        ci += range(q * p, (q + 1) * p)
        rp.append(len(ci))
    m = len(ci)
    cap = np.full(m, 16, np.int32)
    cap[:36] = 16384
    w = si.Workload("stars", E + stars, E, np.array(rp, np.int32), np.array(ci, np.int32), 1, np.full(m, 4, np.int32),
                    np.full(m, 70000, np.int32), cap, 1, -1, 0)
    src = np.repeat(np.arange(E), p - 1).astype(np.int32)
    dst = np.concatenate([[v for v in range(u // p * p, u // p * p + p) if v != u] for u in range(E)]).astype(np.int32)
    return w, (src, dst, np.zeros(len(src) + 1, np.int64), np.zeros(0, np.int64))


# workload -> engine of sim_run, engine of the allocation-free run (None: refused)
CHOICE = [
    # lowest id, one line per cycle: the compact engine at every batch size; the
    # lane engine in LDS where the compact engine's rings exceed the scratch
    ("k4_low_b1_S30", lambda: sweep(si.fat_tree(4, nbytes=256, arb=0), 30, (1,)), "b1", "b1"),
    ("k4_low_b1_S1100", lambda: sweep(si.fat_tree(4, nbytes=256, arb=0), 1100, (1,)), "b1", "lane"),
    ("k6_low_b1_S600", lambda: sweep(si.fat_tree(6, nbytes=128, arb=0), 600, (1,), cap=64), "b1", None),
    # several lines per cycle
    ("k4_low_b2_S100", lambda: sweep(si.fat_tree(4, nbytes=256, arb=0), 100, (1, 2)), "lane", "lane"),
    ("k4_low_b2_S1100", lambda: sweep(si.fat_tree(4, nbytes=256, arb=0), 1100, (1, 2)), "lanehbm", "lane"),
    # round-robin: the route engine, rings in device memory where they do not
    # fit LDS or more scenarios than the chip holds at once
    ("k4_rr_b4_S100", lambda: sweep(si.fat_tree(4, nbytes=256, arb=1), 100, (1, 2, 4)), "route", "route"),
    ("k4_rr_b4_S1700", lambda: sweep(si.fat_tree(4, nbytes=256, arb=1), 1700, (1, 2, 4)), "routehbm", "route"),
    ("k8_rr_b4_S8", lambda: sweep(si.fat_tree(8, nbytes=128, arb=1), 8, (1, 2, 4), cap=32), "routehbm", "routehbm"),
    ("k8_rr_b4_S64", lambda: sweep(si.fat_tree(8, nbytes=128, arb=1), 64, (1, 2, 4), cap=64), "routehbm", None),
    # one large topology
    ("k8_low_S1", lambda: si.fat_tree(8, nbytes=128, arb=0), "b1", "b1"),
    ("k8_low_deep_S1", lambda: replace(si.fat_tree(8, nbytes=128, arb=0), cap=np.full(768, 4096, np.int32)), "b1", None),
    ("k16_S1", lambda: si.fat_tree(16, nbytes=128), "grid", None),
]


# the workloads of the GPU tests of the allocation-free run
@pytest.mark.parametrize("arb,bws,want", [
    (si.ARB_ROUND_ROBIN, (1, 2, 4), {30: ("route", "route"), 1100: ("route", "route"), 1700: ("routehbm", "route")}),
    (si.ARB_LOWEST_ID, (1, 2), {30: ("lane", "lane"), 1100: ("lanehbm", "lane"), 1700: ("lanehbm", "lane")}),
    (si.ARB_LOWEST_ID, (1,), {30: ("b1", "b1"), 1100: ("b1", "lane"), 1700: ("b1", "lane")})])
def test_noalloc_gpu_workloads(plans, arb, bws, want):
    from tests.test_gpu_noalloc_rings import workload
    for S, engines in want.items():
        s = plans.Simulator.from_workload(workload(arb, bws, S))
        assert (launch(plans, s), launch(plans, s, noalloc=True)) == engines, S
        s.close()


@pytest.mark.parametrize("case", CHOICE, ids=[c[0] for c in CHOICE])
def test_engine_choice(plans, case):
    """The engine of sim_run does not depend on the fixed scratch of the
    allocation-free run, which has an engine of its own where it needs one."""
    _, make, run, noalloc = case
    s = plans.Simulator.from_workload(make())
    try:
        assert launch(plans, s) == run
        if noalloc is None:
            with pytest.raises(plans.SimError) as e:
                launch(plans, s, noalloc=True)
            assert e.value.status == plans.SIM_ERR_SIZE
        else:
            assert launch(plans, s, noalloc=True) == noalloc
    finally:
        s.close()


def test_uneven_rings_stay_on_grid(plans):
    """One deep link among shallow ones: the compact engine's rings, all as long
    as the longest, exceed the scratch of the allocation-free run, the grid
    engine's do not."""
    w = si.fat_tree(8, nbytes=128, arb=0)
    w.cap[5] = 4096
    s = plans.Simulator.from_workload(w)
    assert launch(plans, s) == launch(plans, s, noalloc=True) == "grid"
    s.close()


def test_noalloc_takes_what_other_engines_took(plans, monkeypatch):
    """A route-engine load whose rings exceed the scratch runs there on the
    workgroup engine if nothing else could have taken the load and its state,
    12 B per ring entry, fits (latencies beyond the resident engine's 16 bits,
    request slots beyond the lane engine's LDS)."""
    w, txns = deep_stars()
    s = plans.Simulator.from_workload(w)
    s.load_transactions(*txns)
    assert launch(plans, s) == "routehbm"
    assert launch(plans, s, noalloc=True) == "workgroup"
    s.close()
    monkeypatch.setenv("SIMGPU_ENGINE", "lanehbm")
    s = plans.Simulator.from_workload(w)
    with pytest.raises(plans.SimError):
        s.load_transactions(*txns)
    s.close()


@pytest.mark.parametrize("arb,bws,run,short", [(si.ARB_ROUND_ROBIN, (1, 2, 4), "routehbm", "route"),
                                               (si.ARB_LOWEST_ID, (1, 2), "lanehbm", "lane"),
                                               (si.ARB_LOWEST_ID, (1,), "b1", "lane")])
def test_short_of_device_memory(plans, monkeypatch, arb, bws, run, short):
    """Where the device has no room for the rings of a sweep, the load takes the
    engine that keeps them in LDS."""
    w = sweep(si.fat_tree(4, nbytes=256, arb=arb), 1700, bws)
    for most, want in ((0, run), (16 << 20, short)):  # (the rings take 41.8 MB)
        monkeypatch.setenv("SIMGPU_STUB_ALLOC_MAX", str(most))
        s = plans.Simulator.from_workload(w)
        assert launch(plans, s) == want
        assert launch(plans, s, noalloc=True) == short
        s.close()


def test_after_a_load_out_of_memory(plans, monkeypatch):
    """A load that finds no memory reports it, and the next load and run do not
    see its error again."""
    monkeypatch.setenv("SIMGPU_STUB_ALLOC_MAX", str(1 << 20))
    w = sweep(si.fat_tree(8, nbytes=128, arb=1), 8, (1, 2, 4), cap=64)
    ctx = plans.sim_create(w.n_nodes, w.n_endpoints, w.row_ptr, w.col_idx, 8, w.bw, w.lat, w.cap, w.arb)
    with pytest.raises(plans.SimError) as e:
        plans.sim_load_collective(ctx, w.coll, w.bytes)
    assert e.value.status == plans.SIM_ERR_OOM
    plans.sim_load_transactions(ctx, [0], [1], [0, 0], [])
    plans.sim_run(ctx, 0, 1, 1, 1, 1, 0)
    plans.sim_destroy(ctx)


# (tree size, shortest latency and credit delay) -> one wave per workgroup?, workgroups
@pytest.mark.parametrize("k,lo,wave,nb", [(4, 2, True, 32), (4, 64, True, 32), (6, 2, False, 8), (6, 3, True, 32),
                                          (6, 8, True, 99), (8, 2, False, 8), (8, 5, False, 8), (8, 8, True, 208)])
def test_windowed_form(plans, k, lo, wave, nb):
    """Short windows with many sides per workgroup take the multi-wave form."""
    w = si.fat_tree(k, nbytes=128, lat_lo=lo, lat_hi=lo + 3)
    w.credit = np.maximum(w.lat, lo).astype(np.int32)
    w.lat[0] = w.credit[0] = lo
    s = plans.Simulator.from_workload(w)
    assert launch(plans, s) == "grid"
    assert last(plans, "gd_window") == lo
    assert (bool(last(plans, "gd_wave")), last(plans, "gd_nb")) == (wave, nb)
    s.close()


def test_windowed_form_deep_buffers(plans):
    """Eight workgroups' rings beyond LDS: the multi-wave form on 32."""
    w = si.fat_tree(8, nbytes=128, lat_lo=3, lat_hi=5, cap=128)
    w.credit = w.lat.copy()
    s = plans.Simulator.from_workload(w)
    assert launch(plans, s) == "grid"
    assert (last(plans, "gd_wave"), last(plans, "gd_nb")) == (0, 32) and last(plans, "lds_bytes") <= 160 * 1024
    s.close()


def test_windowed_form_gpu_workloads(plans, monkeypatch):
    """The forms that tests/test_gpu_window.py means to run."""
    from tests.test_gpu_window import tree
    for env, want in ({}, 1), ({"SIMGPU_GRID_WINDOW": "multi"}, 0), ({"SIMGPU_GRID_WGS": "1"}, 0), ({"SIMGPU_GRID_WGS": "7"}, 1):
        for v in ("SIMGPU_GRID_WINDOW", "SIMGPU_GRID_WGS"):
            monkeypatch.delenv(v, raising=False)
        for v, x in env.items():
            monkeypatch.setenv(v, x)
        s = plans.Simulator.from_workload(tree(4, 8, 9, 33, 50, 1, 5))
        assert launch(plans, s) == "grid" and last(plans, "gd_wave") == want, env
        s.close()


@pytest.mark.parametrize("arb", [si.ARB_LOWEST_ID, si.ARB_ROUND_ROBIN])
def test_wave_placement_costs(plans, arb):
    """More waves than SIMDs: the shortest by the cost of the loop they run share
    a SIMD (positions j and j + 4 of a workgroup), the longest run alone.  Under
    round-robin, waves of several lines per cycle run the shift loop, not the
    chain loop."""
    S = 4500
    w = si.torus2d(4, 4, n_scenarios=S, seed=12, bws=(1, 4), depths=(8, 12, 16, 24, 32, 48, 64), nbytes=128 * 16 * 8,
                   arb=arb)
    s = plans.Simulator.from_workload(w)
    assert launch(plans, s) == "wave" and last(plans, "wv_chain") == 1
    bw, cap = w.bw[::w.n_links], w.cap[::w.n_links].astype(float)
    per = np.where(bw == 1, 0.27, 0.82 if arb == si.ARB_LOWEST_ID else 1.2)
    cost = (1.0 / bw + 4.0 / cap) * per  # (lines on the busiest link: the same in every scenario)
    nblk, wpb, W, G = (last(plans, "wv_" + v) for v in ("nblk", "wpb", "W", "G"))
    blk = np.ctypeslib.as_array(plans.lib().stub_blk_wave(), (nblk, wpb))
    sc = np.ctypeslib.as_array(plans.lib().stub_wv_sc(), (W * G,)).reshape(W, G)
    assert 4 < wpb <= 8 and 1024 < W <= 2048
    wave = np.array([cost[v[v >= 0]].max() for v in sc])  # as long as its longest scenario
    alone, shared = [], []
    for b in blk:
        for j in range(4):
            if b[j] < 0:
                continue
            pair = [b[j]] + [b[q] for q in (j + 4,) if q < wpb and b[q] >= 0]
            (shared if len(pair) == 2 else alone).extend(pair)
    assert sorted(alone + shared) == list(range(W))
    assert wave[alone].min() >= wave[shared].max() - 1e-9
    s.close()


def test_chain_gpu_workloads(plans, monkeypatch):
    """The loops that tests/test_gpu_chain.py means to run: the chain loops, the
    shift loop where it is asked for, the general loops on other graphs."""
    def loop(w, txns=None):
        s = plans.Simulator.from_workload(w)
        if txns is not None:
            s.load_transactions(*txns)
        assert launch(plans, s) == "wave"
        s.close()
        return "chain" if last(plans, "wv_chain") else "shift" if last(plans, "wv_lineup") else "general"

    ring = []
    for arb in (0, 1):
        for dep in (si.DEP_LINE, si.DEP_CHUNK):
            for coll in (si.COLL_RING_ALLREDUCE, si.COLL_RING_ALLGATHER):
                ring.append(replace(si.torus2d(4, 4, n_scenarios=14, seed=31, bws=(1, 2, 4), depths=(1, 2, 3, 5, 16, 33),
                                               nbytes=128 * 16 * 6, arb=arb, coll=coll), dep=dep))
            for p, b, coll in ((3, 1, si.COLL_DIRECT_ALLREDUCE), (8, 4, si.COLL_RHD_ALLREDUCE), (7, 1, si.COLL_DBT_ALLREDUCE),
                               (5, 2, si.COLL_RING_ALLREDUCE)):
                ring.append(replace(si.full_mesh(p, b=b, L=6, cap=4, coll=coll, nbytes=128 * 6 * p, arb=arb), dep=dep))
        for coll in (si.COLL_RING_ALLREDUCE,) + ((si.COLL_RHD_ALLREDUCE,) if arb == 0 else ()):  # stopped by the guard
            w = si.torus2d(4, 2, n_scenarios=12, seed=51, bws=(2,), depths=(2, 5, 16), nbytes=128 * 8 * 24, arb=arb, coll=coll)
            ring.append(replace(w, order=si.gray_torus_order(4, 2)) if coll == si.COLL_RHD_ALLREDUCE else w)
    assert {loop(w) for w in ring} == {"chain"}
    src, dst = np.arange(5, dtype=np.int32), (np.arange(5, dtype=np.int32) + 1) % 5
    assert loop(si.full_mesh(5, b=2, L=3, cap=3, nbytes=128 * 5),
                (src, dst, np.zeros(6, np.int64), np.zeros(0, np.int64))) == "chain"
    same = si.torus2d(4, 4, n_scenarios=40, seed=8, bws=(1, 2, 4), depths=(4, 16, 40), nbytes=128 * 16 * 40)
    for env, want in (("", "chain"), ("shift", "shift"), ("general", "general")):
        monkeypatch.setenv("SIMGPU_WAVE_LOOP", env)
        assert loop(same) == want
    monkeypatch.delenv("SIMGPU_WAVE_LOOP")
    from tests.test_gpu_chain import EIGHT_LINES
    for X, Y, coll in EIGHT_LINES:
        assert loop(si.torus2d(X, Y, n_scenarios=9, seed=61, bws=(5, 8), depths=(9, 24, 40), nbytes=128 * X * Y * 14, arb=1,
                               coll=coll)) == "general"
    rp, ci, three = np.array([0, 1, 2, 3], np.int32), np.array([1, 2, 0], np.int32), np.full(3, 8, np.int32)
    w = si.Workload("ring3", 3, 3, rp, ci, 1, three, three, three, 1, -1, 0)
    assert loop(w, (np.array([0, 1, 2], np.int32), np.array([2, 0, 1], np.int32), np.zeros(4, np.int64),
                    np.zeros(0, np.int64))) == "general"

"""Compact engine: ranges with more predecessors than its registers cache
(direct all-reduces on meshes of more than nine endpoints, random DAGs), next to
ranges with few and none -- parity with the CPU oracle in both dependency modes
and both arbitrations, over several scenarios."""
from __future__ import annotations

import numpy as np
import pytest

import sim_inputs as si
from tests.test_gpu_parity import check_engine, simmod, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arb", [0, 1])
@pytest.mark.parametrize("dep", [si.DEP_LINE, si.DEP_CHUNK])
@pytest.mark.parametrize("p,per", [(9, 5), (10, 1), (17, 3), (18, 4), (26, 2)])
def test_direct(simmod, oracle_lib, p, per, dep, arb):
    w = si.full_mesh(p, b=1, L=4, cap=3, coll=si.COLL_DIRECT_ALLREDUCE, nbytes=128 * per * p, arb=arb)
    m = w.n_links
    rng = np.random.default_rng(p)
    w.n_scenarios = 2
    w.lat = np.concatenate([np.full(m, 5), rng.integers(1, 12, m)]).astype(np.int32)  # in step, and not
    w.bw = np.ones(2 * m, np.int32)
    w.cap = np.repeat([16, 2], m).astype(np.int32)
    w.dep = dep
    assert check_engine(simmod, oracle_lib, w, "b1", must_run=True) == 2


@pytest.mark.parametrize("n_preds", [7, 8, 9, 17, 40])
def test_predecessors(simmod, oracle_lib, n_preds):
    """Single-line ranges, each waiting on up to n_preds flows."""
    rng = np.random.default_rng(700 + n_preds)
    p, n = 8, 300
    src = rng.integers(0, p, n).astype(np.int32)
    dst = ((src + rng.integers(1, p, n)) % p).astype(np.int32)
    pptr, pidx = [0], []
    for x in range(n):
        k = min(x, int(rng.integers(0, n_preds + 1)))
        pidx += sorted(int(v) for v in rng.choice(x, size=k, replace=False)) if k else []
        pptr.append(len(pidx))
    w = si.full_mesh(p, b=1, L=3, cap=3, nbytes=128)
    check_engine(simmod, oracle_lib, w, "b1", txns=(src, dst, np.array(pptr, np.int64), np.array(pidx, np.int64)),
                 must_run=True)

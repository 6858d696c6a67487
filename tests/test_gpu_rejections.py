"""Uniform proposals that reject many times (needs an MI355X): rejected trials are drawn again within a
pass of the walk kernel, up to the step's trial cap.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from tests._gpu import GpuGraph, assert_parity, fw_plan, gpu_walk, parity
from tests.test_gpu_launch_cost import Walks, best_us
from tests.test_gpu_parity import MP

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
LOGICS = {
    "node2vec": oracle.Logic(kind=oracle.NODE2VEC, weighted=True, p=0.25, q=4.0),
    "node2vec_unweighted": oracle.Logic(kind=oracle.NODE2VEC, weighted=False, p=4.0, q=0.25),
    "node2vec_unweighted_return": oracle.Logic(kind=oracle.NODE2VEC, weighted=False, p=0.25, q=4.0),
    "secondpr_unweighted": oracle.Logic(kind=oracle.SECOND_PR, weighted=False, gamma=0.5),
    "secondpr": oracle.Logic(kind=oracle.SECOND_PR, weighted=True, gamma=0.9),
    "metapath": MP,
    "metapath_unweighted": oracle.Logic(kind=oracle.METAPATH, weighted=False, schema=MP.schema),
}


@pytest.mark.parametrize("n", [1, 61, 5000])
@pytest.mark.parametrize("cap", [1, 2, 3, 4, 5, 64, 65, 1024])
@pytest.mark.parametrize("logic", sorted(LOGICS))
def test_rejected_trials(logic, cap, n):
    """Waves of one walker, a few and many; caps around the trials of a pass and where the wave takes
    over: equal to the oracle, with the index and by search, with each board, with and without
    counters, and as many trials counted either way."""
    print("rejections", logic, cap, n, flush=True)
    g = synth.rmat(10, 12 << 10, seed=4, nlabels=5)
    heavy = (np.arange(g["ne"]) * 7 + g["col"]) % 53 == 0
    if logic == "metapath":  # (other logics' graphs have equal weights in both directions)
        g["h"] = np.where(heavy, g["h"] * np.float32(50), g["h"]).astype(np.float32)
    lg = LOGICS[logic]
    starts = synth.uniform_starts(g["nv"], n, 5)
    L = 12
    for index, bound in ((True, 0), (False, 0)) + (((True, 1),) if "node2vec" in logic else ()) + \
            (((True, 2), (False, 2)) if "metapath" not in logic else ()):
        pl = oracle.Plan(rho=0.3, rjs_cap=cap, bound=bound)
        gg = GpuGraph(g, index=index)
        try:
            p0, l0, st = gpu_walk(gg, lg, pl, oracle.RJS_ONLY, starts, L, 11)
            p1, l1, _ = gpu_walk(gg, lg, pl, oracle.RJS_ONLY, starts, L, 11, counters=False)
        finally:
            gg.close()
        np.testing.assert_array_equal(p1, p0)
        np.testing.assert_array_equal(l1, l0)
        ora = oracle.walk(oracle.Graph(g), lg, pl, oracle.RJS_ONLY, starts, L, 11)
        rep = parity(p0, l0, ora)
        assert_parity(rep)
        if rep["mismatch_walkers"] == 0:
            for c in ("steps", "rjs_steps", "rvs_steps", "rjs_fallbacks", "rjs_trials", "ended_early", "alg_bytes"):
                assert st[c] == ora.counters[c], (c, index, bound)


def test_time_of_rejections():
    """Node2Vec with p = 1/4, q = 4: walks by uniform proposals, which reject most, take less than 2.1
    times as long as by proposals from records (with a pass of the kernel for each trial: 2.35 times)."""
    g = synth.rmat(16, 16 << 16, seed=3)
    gg = GpuGraph(g, index=True, alias=True)
    lg = LOGICS["node2vec"]
    try:
        uni = Walks(gg, lg, fw_plan(oracle.Plan(rho=0.4, bound=1)), fw.FW_AUTO, 109000, 52)
        rec = Walks(gg, lg, fw_plan(oracle.Plan(rho=0.4, bound=2, proposal=1)), fw.FW_AUTO, 109000, 52)
        t0, t1 = best_us(rec), best_us(uni)
        print("us", t0, t1, t1 / t0, flush=True)
        assert t1 < 2.1 * t0, (t0, t1)
    finally:
        gg.close()

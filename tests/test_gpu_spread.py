"""Launches of fewer walkers than the grid has lanes (needs an MI355X).

Such a launch spreads its walkers over all waves, a few lanes of each: walker counts around
the multiples of the wave count (the first lane of every wave, one lane more, all lanes, one
walker past the grid's lanes) must give the oracle's walks.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from tests._gpu import GpuGraph, assert_parity, fw_plan, parity
from tests.test_gpu_batch import Batch
from tests.test_gpu_parity import N2V, STRATS, _run_both

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
GRID = 2  # 8 waves, 512 lanes


@pytest.fixture(scope="module")
def g9():
    return synth.rmat(9, 8 << 9, seed=1)


@pytest.fixture(scope="module")
def gg9(g9):
    gg = GpuGraph(g9, index=True, alias=True)
    yield gg
    gg.close()


@pytest.mark.parametrize("grid", [0, GRID])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 17, 504, 505, 511, 512, 513, 1300])
@pytest.mark.parametrize("strategy,proposal", [("rvs", 0), ("auto", 0), ("auto", 1)])
def test_walker_counts_around_the_grid(gg9, g9, n, grid, strategy, proposal):
    print("spread", n, grid, strategy, proposal, flush=True)
    starts = synth.uniform_starts(g9["nv"], n, 5)
    pl = oracle.Plan(rho=2.0 if proposal == 0 else 0.4, proposal=proposal, bound=2 if proposal else 0)
    p, ln, _, ora = _run_both(gg9, g9, N2V, pl, STRATS[strategy], starts, 9, 21, grid=grid)
    assert_parity(parity(p, ln, ora))


@pytest.mark.parametrize("sizes", [(1,), (3, 0, 5), (1, 7, 500, 4), (513, 1, 200)])
def test_batch_walker_counts_around_the_grid(gg9, g9, sizes):
    """The queries of a batch share the waves' lanes; each equals its own fw_walk."""
    print("spread batch", sizes, flush=True)
    n = np.array(sizes, np.int64)
    L = np.array([5 + 3 * i for i in range(len(sizes))], np.int32)
    off = np.concatenate([[0], np.cumsum(n)[:-1]]).astype(np.int64)
    qd = {"n": n, "L": L, "seed": 40 + np.arange(len(sizes)), "start_off": off, "len_off": off,
          "out_off": np.concatenate([[0], np.cumsum(n * (L.astype(np.int64) + 1))[:-1]]).astype(np.int64),
          "starts": synth.uniform_starts(g9["nv"], int(n.sum()), 6)}
    pl = oracle.Plan(rho=2.0)
    b = Batch(gg9, qd, [fw.fw_logic_node2vec(2.0, 0.5, True)] * len(sizes), fw_plan(pl, grid=GRID), fw.FW_AUTO)
    try:
        fw.fw_batch_launch(b.h)
        for i in range(len(sizes)):
            p, ln = b.query(i)
            s = qd["starts"][off[i]:off[i] + n[i]]
            ora = oracle.walk(oracle.Graph(g9), oracle.Logic(kind=oracle.NODE2VEC, weighted=True, p=2.0, q=0.5), pl,
                              oracle.AUTO, s, int(L[i]), int(qd["seed"][i]))
            bad = np.flatnonzero((p != ora.paths).any(axis=1) | (ln != ora.lengths))
            assert all((ora.margins[w] < 1e-6).any() for w in bad), (i, bad[:5])
    finally:
        b.close()

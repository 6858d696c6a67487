"""What creating a graph and building its tables read from it (needs an MI355X): rows that start,
end and change anywhere among the 64 entries that a wave takes at a time, long runs of empty
rows, rows much longer than the others.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests._gpu import GpuGraph, assert_parity, gpu_walk, parity

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu


def _rows(lens, nv, seed=3):
    """Rows of the given lengths (the others empty) with random ascending neighbours."""
    rng = np.random.default_rng(seed)
    row_ptr = np.zeros(nv + 1, np.int64)
    row_ptr[1 : 1 + len(lens)] = lens
    row_ptr = np.cumsum(row_ptr)
    col = np.concatenate([np.sort(rng.choice(nv, n, replace=False)) for n in lens] or [np.zeros(0)]).astype(np.int32)
    h = rng.integers(1, 9, len(col)).astype(np.float32)
    return {"nv": nv, "ne": len(col), "row_ptr": row_ptr, "col": col, "h": h}


def _symmetric(leaves, gap):
    """A star whose leaves lie `gap` vertices apart, and a path through them."""
    ids = [gap * (i + 1) for i in range(leaves)]
    edges = [(0, i) for i in ids] + [(ids[i], ids[i + 1]) for i in range(0, leaves - 1, 2)]
    g = synth.csr_from_edges(ids[-1] + gap, edges)
    src = np.repeat(np.arange(g["nv"]), np.diff(g["row_ptr"]))
    lo, hi = np.minimum(src, g["col"]), np.maximum(src, g["col"])
    g["h"] = (1 + (lo * 7 + hi * 13) % 5).astype(np.float32)
    return g


def _drop(g, k):
    out = dict(g, ne=g["ne"] - 1, col=np.delete(g["col"], k), h=np.delete(g["h"], k), row_ptr=g["row_ptr"].copy())
    out["row_ptr"][np.searchsorted(g["row_ptr"], k, side="right") :] -= 1
    return out


@pytest.mark.parametrize("leaves,gap", [(1, 1), (31, 1), (63, 3), (64, 1), (129, 70), (3000, 7), (500, 5000)])
def test_symmetry_is_seen(leaves, gap):
    """fw_graph_info's `symmetric` of a symmetric graph, of one that lacks one entry (the first, one
    in the middle, the last) and of one with a different weight on one direction."""
    g = _symmetric(leaves, gap)

    def symmetric(x):
        gg = GpuGraph(x, preprocess=False)
        try:
            return bool(fw.fw_graph_info(gg.handle)[3])
        finally:
            gg.close()

    assert symmetric(g)
    for k in {0, g["ne"] // 2, g["ne"] - 1}:
        assert not symmetric(_drop(g, k))
        h = g["h"].copy()
        h[k] += 1
        assert not symmetric(dict(g, h=h))


def test_directed_cycle_is_not_symmetric():
    g = synth.csr_from_edges(4, [(0, 1), (1, 2), (2, 3), (3, 0)], symmetric=False)
    gg = GpuGraph(g, preprocess=False)
    try:
        assert not fw.fw_graph_info(gg.handle)[3]
    finally:
        gg.close()


@pytest.mark.parametrize("at", [1, 63, 64, 65, 255, 256, 4095])
def test_rows_must_ascend(at):
    """Equal and falling neighbours are refused wherever they are; a fall at a row's start is none."""
    g = _rows([at, 4096 - at, 40], 9000)
    GpuGraph(g).close()
    for k in (max(1, at - 1), at + 1, 4095 if at < 4094 else 4097):
        if k in g["row_ptr"]:
            continue
        for c in (g["col"][k - 1], max(0, g["col"][k - 1] - 1)):
            bad = g["col"].copy()
            bad[k] = c
            with pytest.raises(fw.FlexiWalkError) as e:
                GpuGraph(dict(g, col=bad))
            assert e.value.code == fw.FW_E_INVALID


@pytest.mark.parametrize("where", [0, 77, -1])
@pytest.mark.parametrize("bad", ["col_low", "col_high", "nan", "inf", "negative"])
def test_bad_entries_are_refused(bad, where):
    g = _rows([50, 1, 80], 300)
    col, h = g["col"].copy(), g["h"].copy()
    if bad.startswith("col"):
        col[where] = -1 if bad == "col_low" else 300
    else:
        h[where] = {"nan": np.nan, "inf": np.inf, "negative": -1.0}[bad]
    with pytest.raises(fw.FlexiWalkError) as e:
        GpuGraph(dict(g, col=col, h=h))
    assert e.value.code == fw.FW_E_INVALID


@pytest.mark.parametrize("leaves,gap", [(1, 1), (64, 1), (129, 70), (3000, 7), (500, 5000)])
def test_index_holds_every_entry(leaves, gap):
    """Walks by the index equal walks that search the rows."""
    g = _symmetric(leaves, gap)
    starts = np.repeat(np.array([0, gap], np.int32), 700)
    lg, pl = oracle.Logic(kind=oracle.NODE2VEC, weighted=True, p=4.0, q=0.25), oracle.Plan(rho=0.01)
    out = []
    for index in (False, True):
        gg = GpuGraph(g, index=index)
        try:
            p, ln, _ = gpu_walk(gg, lg, pl, oracle.AUTO, starts, 20, 5)
            out.append((np.asarray(p), np.asarray(ln)))
        finally:
            gg.close()
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("weights", ["random", "equal", "zeros", "one_heavy", "none"])
@pytest.mark.parametrize("lens", [[1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64], [65, 1, 127, 128, 129, 64, 1000],
                                  [8191, 8192, 8193, 2, 66], [10241, 3, 32768, 32769, 70]])
def test_alias_tables_of_row_lengths(lens, weights):
    """Rows built whole by a few lanes, by a wave's sums, by a block's: equal to the sequential sweep."""
    g = _rows(lens, 40000)
    if weights == "equal":
        g["h"][:] = 3.0
    elif weights == "zeros":
        g["h"][np.arange(g["ne"]) % 3 != 1] = 0.0
        g["h"][g["row_ptr"][1] : g["row_ptr"][2]] = 0.0
    elif weights == "one_heavy":
        g["h"][g["row_ptr"][1 : len(lens) + 1] - 1] = 1e6
    elif weights == "none":
        g["h"] = None
    gg = GpuGraph(g, alias=True)
    try:
        thr, al = fw.fw_graph_export_alias(gg.handle, gg.ne)
    finally:
        gg.close()
    othr, oal = oracle.Graph(g).alias()
    np.testing.assert_array_equal(al, oal)
    np.testing.assert_array_equal(thr, othr)


def test_graphs_one_after_another():
    """Graphs of changing sizes from several threads at once, created, built, walked and destroyed
    in turn (their memory is kept for the next ones, at most 8 GiB of it): every walk equals the
    oracle's, whatever the blocks held before."""
    import threading

    lg, pl = oracle.Logic(kind=oracle.NODE2VEC, weighted=True, p=4.0, q=0.25), oracle.Plan(rho=1.0, proposal=1)
    cases = []
    for scale, seed in ((13, 1), (15, 2), (14, 3), (15, 4)):
        g = synth.rmat(scale, 12 << scale, seed=seed)
        starts = np.arange(0, g["nv"], 97, dtype=np.int32)
        cases.append((g, starts, oracle.walk(oracle.Graph(g), lg, pl, oracle.AUTO, starts, 12, seed)))
    free0 = torch.cuda.mem_get_info()[0]
    done = []

    def work(first):
        for i in range(10):
            g, starts, want = cases[(first + i) % len(cases)]
            gg = GpuGraph(g, index=bool(i % 2), alias=True)
            try:
                p, ln, _ = gpu_walk(gg, lg, pl, oracle.AUTO, starts, 12, 1 + (first + i) % len(cases))
            finally:
                gg.close()
            done.append(parity(p, ln, want))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(done) == 30
    for rep in done:
        assert_parity(rep)
    assert free0 - torch.cuda.mem_get_info()[0] < (9 << 30)

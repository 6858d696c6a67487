"""What a launch costs beside its walks (needs an MI355X): counters and work hand-out go through
one address each, which must not set the time of a short launch.  Every bound compares two ways
to take the same walks on the same device, with room for noise.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests._gpu import GpuGraph, fw_logic, fw_plan
from tests.test_gpu_parity import N2V, MP

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def best_us(f, reps=12):
    """The fastest of `reps` calls by events, after one that warms up."""
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


class Walks:
    """fw_walk of n walkers x L steps into buffers of its own."""

    def __init__(self, gg, lg, plan, strategy, n, L, counted=False, seed=5):
        self.starts = torch.from_numpy(synth.uniform_starts(gg.nv, n, 2)).to(DEV)
        self.paths = torch.full((n, L + 1), -7, dtype=torch.int32, device=DEV)
        self.lengths = torch.full((n,), -7, dtype=torch.int32, device=DEV)
        self.stats = torch.zeros(fw.FW_NSTATS, dtype=torch.int64, device=DEV) if counted else None
        self.args = (gg.handle, fw_logic(lg), plan, strategy, self.starts, n, L, seed, self.paths, self.lengths,
                     self.stats)

    def __call__(self):
        fw.fw_walk(*self.args)

    def out(self):
        torch.cuda.synchronize()
        return self.paths.cpu().numpy(), self.lengths.cpu().numpy()


def same(a, b):
    for x, y in zip(a.out(), b.out()):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("strategy", ["auto", "rvs"])
def test_counters_of_a_short_launch(strategy):
    """One step of 60000 walkers with device counters takes less than three times as long as without
    (with an add per wave and counter: 4 to 8 times)."""
    print("counters", strategy, flush=True)
    g = synth.rmat(12, 24 << 12, seed=3, nlabels=5)
    gg = GpuGraph(g, index=True)
    try:
        lg = MP
        pl = fw_plan(oracle.Plan(rho=0.4, d_lo=32))
        s = fw.FW_AUTO if strategy == "auto" else fw.FW_RVS_ONLY
        plain, counted = Walks(gg, lg, pl, s, 60000, 1), Walks(gg, lg, pl, s, 60000, 1, counted=True)
        t0, t1 = best_us(plain), best_us(counted)
        same(plain, counted)
        st = dict(zip(fw.STAT_NAMES, counted.stats.tolist()))
        assert st["steps"] == 13 * int(plain.lengths.sum().item())  # 13 launches add up
        assert t1 < 3 * t0, (t0, t1)
    finally:
        gg.close()


@pytest.mark.parametrize("n", [6000, 30001, 300000])
def test_one_step_reservoir_walks(n):
    """FW_RVS_ONLY walks of one step take less than twice as long as the same walks by the kernel of
    the other strategies, which hands walkers out without a counter (with a few walkers per add of
    every wave: 2.5 to 3.5 times)."""
    print("one step", n, flush=True)
    g = synth.rmat(17, 16 << 17, seed=3)
    gg = GpuGraph(g)
    try:
        other = Walks(gg, N2V, fw_plan(oracle.Plan(d_lo=1 << 30)), fw.FW_DEGREE_SELECT, n, 1)
        rvs = Walks(gg, N2V, fw_plan(oracle.Plan()), fw.FW_RVS_ONLY, n, 1)
        t0, t1 = best_us(other), best_us(rvs)
        same(other, rvs)
        assert t1 < 2 * t0, (t0, t1)
    finally:
        gg.close()


@pytest.mark.parametrize("strategy,hub", [("auto", False), ("auto", True), ("rvs", False), ("rvs", True)])
def test_lds_cap_past_its_room(strategy, hub):
    """A plan's lds_cap above what finds room beside the kernels' other needs costs no time (with
    fewer resident blocks for it: 2.5 times) and changes no walk."""
    print("lds_cap", strategy, hub, flush=True)
    g = synth.rmat(15, 16 << 15, seed=3)
    gg = GpuGraph(g)
    try:
        s = fw.FW_AUTO if strategy == "auto" else fw.FW_RVS_ONLY
        pl = oracle.Plan(d_lo=1 << 30, hub_deg=1024 if hub else 0, hub_lanes=256 if hub else 64)
        runs = [Walks(gg, N2V, fw_plan(pl, lds_cap=cap), s, 30000, 20) for cap in (512, 2048, 8192)]
        t = [best_us(r, 6) for r in runs]
        for r in runs[1:]:
            same(runs[0], r)
        assert max(t[1:]) < 1.3 * t[0], t
    finally:
        gg.close()


@pytest.mark.parametrize("over", [1.01, 1.2])
def test_a_few_more_walkers_than_lanes(over):
    """A launch of a fifth more walkers than the kernel has lanes takes less than 1.5 times one that
    they hold (with the fifth handed out by the counter: 1.6 to 1.7 times)."""
    print("over", over, flush=True)
    g = synth.rmat(14, 16 << 14, seed=3, nlabels=5)
    gg = GpuGraph(g, label_alias=True)
    try:
        lanes = torch.cuda.get_device_properties(0).multi_processor_count * 4 * 4 * 64
        pl = fw_plan(oracle.Plan(rho=0.4, proposal=2))
        held = Walks(gg, MP, pl, fw.FW_AUTO, lanes - 64, 40)
        more = Walks(gg, MP, pl, fw.FW_AUTO, int(lanes * over), 40)
        t0, t1 = best_us(held), best_us(more)
        print("us", t0, t1, flush=True)
        assert t1 < 1.5 * t0, (t0, t1)
    finally:
        gg.close()


def _with_zero_rows(scale, rows, starts):
    """R-MAT of 16 draws per vertex whose edges weigh 0 at the first start that has any (rows = 1) or at
    a share of the vertices (rows < 1)."""
    g = synth.rmat(scale, 16 << scale, seed=3, nlabels=5)
    src = np.repeat(np.arange(g["nv"]), np.diff(g["row_ptr"]))
    has = np.flatnonzero(np.diff(g["row_ptr"]) > 0)
    zero = np.zeros(g["nv"], bool)
    zero[starts[np.isin(starts, has)][0] if rows == 1 else has[:: int(1 / rows)] if rows else []] = True
    g["h"] = np.where(zero[src] | zero[g["col"]], np.float32(0), g["h"]).astype(np.float32)
    return g


@pytest.mark.parametrize("rows", [1, 0.01])
def test_few_rows_of_zero_weight(rows):
    """Walks that meet a row whose weights are all 0 go to eRVS; one such row, or one in a hundred,
    does not slow a launch that is compiled without eRVS to more than 1.5 times (with the parked
    walks found through the counter: 2.3 to 2.6 times)."""
    print("zero rows", rows, flush=True)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 4 * 4 * 64 * 3 // 2
    pl = fw_plan(oracle.Plan(rho=0.4, proposal=1, bound=2))
    t = []
    for r in (0, rows):
        gg = GpuGraph(_with_zero_rows(17, r, synth.uniform_starts(1 << 17, n, 2)), index=True, alias=True)
        try:
            w = Walks(gg, N2V, pl, fw.FW_AUTO, n, 5)
            t.append(best_us(w))
            if r:
                ref = oracle.walk(oracle.Graph(gg.g), N2V, oracle.Plan(rho=0.4, proposal=1, bound=2), oracle.AUTO,
                                  w.starts[:2000].cpu().numpy(), 5, 5)
                p, ln = w.out()
                np.testing.assert_array_equal(p[:2000], ref.paths)
                np.testing.assert_array_equal(ln[:2000], ref.lengths)
        finally:
            gg.close()
    print("us", t, flush=True)
    assert t[1] < 1.5 * t[0], t


def test_rows_without_the_label():
    """MetaPath walks with uniform proposals reach the trial cap at every row without the wanted label:
    launches above the kernel's lanes take no more than 1.5 times those that they hold (with the walks
    of such rows parked: 4 to 5 times)."""
    g = synth.rmat(14, 2 << 14, seed=3, nlabels=5)
    gg = GpuGraph(g)
    try:
        lanes = torch.cuda.get_device_properties(0).multi_processor_count * 4 * 4 * 64
        pl = fw_plan(oracle.Plan(rho=0.4, rjs_cap=64))
        t = [best_us(Walks(gg, MP, pl, fw.FW_RJS_ONLY, n, 1)) for n in (lanes - 64, lanes * 11 // 10)]
        print("us", t, flush=True)
        assert t[1] < 1.5 * t[0], t
    finally:
        gg.close()


def test_short_reservoir_walks():
    """FW_RVS_ONLY walks of a few short rows each take no longer than 1.12 times the same walks by the
    kernel of the other strategies (with an add to the counter per finished walk: 1.3 times)."""
    g = synth.rmat(15, 8 << 15, seed=3, nlabels=5)
    gg = GpuGraph(g)
    try:
        other = Walks(gg, MP, fw_plan(oracle.Plan(d_lo=1 << 30)), fw.FW_DEGREE_SELECT, 180000, 5)
        rvs = Walks(gg, MP, fw_plan(oracle.Plan()), fw.FW_RVS_ONLY, 180000, 5)
        t0, t1 = best_us(other), best_us(rvs)
        same(other, rvs)
        print("us", t0, t1, flush=True)
        assert t1 < 1.12 * t0, (t0, t1)
    finally:
        gg.close()


def test_first_order_pagerank():
    """Second-order PageRank with gamma = 0 weighs all neighbours alike, as Node2Vec with p = q = 1: with
    uniform proposals its walks take no longer than 1.12 times (spread over twice the waves: 1.24)."""
    g = synth.rmat(12, 16 << 12, seed=3)
    gg = GpuGraph(g, index=True)
    try:
        pl = fw_plan(oracle.Plan(rho=0.4))
        n2v = oracle.Logic(kind=oracle.NODE2VEC, weighted=True, p=1.0, q=1.0)
        pr = oracle.Logic(kind=oracle.SECOND_PR, weighted=True, gamma=0.0)
        t0, t1 = (best_us(Walks(gg, lg, pl, fw.FW_AUTO, 25000, 40)) for lg in (n2v, pr))
        print("us", t0, t1, flush=True)
        assert t1 < 1.12 * t0, (t0, t1)
    finally:
        gg.close()


@pytest.mark.parametrize("first", [0, 1])
def test_first_order_pagerank_in_a_mixed_batch(first):
    """A batch with one small gamma = 0 query takes no longer than 1.1 times its other queries alone,
    wherever that query stands in the table."""
    g = synth.rmat(16, 16 << 16, seed=3)
    gg = GpuGraph(g, index=True)
    try:
        pl, n, L = fw_plan(oracle.Plan(rho=0.4)), 60000, 40
        starts = torch.from_numpy(synth.uniform_starts(g["nv"], n + 1, 2)).to(DEV)
        paths = torch.empty((n + 1) * (L + 1), dtype=torch.int32, device=DEV)
        lengths = torch.empty(n + 1, dtype=torch.int32, device=DEV)
        small = fw.fw_query(fw.fw_logic_second_pr(0.0, True), 1, L, 5, n, n * (L + 1), n)
        big = fw.fw_query(fw.fw_logic_second_pr(0.5, True), n, L, 6, 0, 0, 0)
        t = []
        for qs in ([big], [small, big] if first else [big, small]):
            b = fw.fw_batch_create(gg.handle, qs, pl, fw.FW_AUTO, starts, paths, lengths)
            t.append(best_us(lambda: fw.fw_batch_launch(b)))
            fw.fw_batch_destroy(b)
        print("us", t, flush=True)
        assert t[1] < 1.1 * t[0], t
    finally:
        gg.close()

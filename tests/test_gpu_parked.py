"""Walks that meet an eRVS step in a launch compiled without eRVS (needs an MI355X): they are parked
and run on by a second launch.  Launch sizes follow the device, and the counted run shows that
there were such steps.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests._gpu import GpuGraph, assert_parity, fw_logic, fw_plan, gpu_walk, parity
from tests.test_gpu_parity import N2V

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
PR2 = oracle.Logic(kind=oracle.SECOND_PR, weighted=True, gamma=0.2)
LOGICS = {"node2vec": N2V, "secondpr": PR2}


def lanes():
    """Walkers that the form with the scan holds at once (four waves per SIMD); above, launches whose
    plan sends every ordinary step to eRJS leave the scan out."""
    return torch.cuda.get_device_properties(0).multi_processor_count * 4 * 4 * 64


def few_zero_rows():
    """Scale 12 with all edges at two vertices of weight 0 (fewer rows than one in 1024)."""
    g = synth.rmat(12, 8 << 12, seed=4)
    src = np.repeat(np.arange(g["nv"]), np.diff(g["row_ptr"]))
    zero = np.flatnonzero(np.diff(g["row_ptr"]) > 0)[[3, 900]]
    g["h"] = np.where(np.isin(src, zero) | np.isin(g["col"], zero), np.float32(0), g["h"]).astype(np.float32)
    return g, zero


def heavy_edges():
    """Scale 9 with a few edges 10^4 times the others: uniform trials run into the cap."""
    g = synth.rmat(9, 8 << 9, seed=4)
    src = np.repeat(np.arange(g["nv"]), np.diff(g["row_ptr"]))
    lo, hi = np.minimum(src, g["col"]), np.maximum(src, g["col"])
    g["h"] = np.where((lo * 31 + hi * 17) % 97 == 0, g["h"] * np.float32(1e4), g["h"]).astype(np.float32)
    return g


@pytest.mark.parametrize("logic", sorted(LOGICS))
@pytest.mark.parametrize("size", [1.01, 1.3, 4.1])
@pytest.mark.parametrize("case", ["zero_rows", "cap"])
def test_parked_walks_run_on(case, size, logic):
    """Some walks parked at their start (rows of zeros) or on their way (trial cap): equal to the counted
    launch, which has the scan, on every walker, and to the oracle on the first 2000."""
    print("parked", case, size, logic, flush=True)
    n, L, lg = int(lanes() * size) + 7, 7, LOGICS[logic]
    g, zero = few_zero_rows() if case == "zero_rows" else (heavy_edges(), None)
    gg = GpuGraph(g, index=True, alias=True)
    try:
        starts = synth.uniform_starts(g["nv"], n, 9)
        if case == "zero_rows":
            starts[5::37] = zero[0]
            starts[n - 300:] = zero[1]  # whole waves of them
            pl, strategy = oracle.Plan(rho=0.3, proposal=1), oracle.AUTO
        else:
            pl, strategy = oracle.Plan(rho=0.3, rjs_cap=64), oracle.RJS_ONLY
        p0, l0, st = gpu_walk(gg, lg, pl, strategy, starts, L, 3)
        p1, l1, _ = gpu_walk(gg, lg, pl, strategy, starts, L, 3, counters=False)
        assert st["rjs_fallbacks"] + st["rvs_steps"] > 0 if case == "cap" else (l0[starts == zero[0]] == 0).all()
        np.testing.assert_array_equal(p1, p0)
        np.testing.assert_array_equal(l1, l0)
        assert_parity(parity(p1[:2000], l1[:2000],
                             oracle.walk(oracle.Graph(g), lg, pl, strategy, starts[:2000], L, 3)))
    finally:
        gg.close()


@pytest.mark.parametrize("case", ["zero_rows", "cap"])
def test_parked_walks_of_a_batch(case):
    """The same in a batch of a small and a large query, launched and replayed from its HIP graph."""
    print("parked batch", case, flush=True)
    g, zero = few_zero_rows() if case == "zero_rows" else (heavy_edges(), None)
    gg = GpuGraph(g, index=True, alias=True)
    try:
        n = [5, int(lanes() * 1.1)]
        L = [9, 6]
        starts = synth.uniform_starts(g["nv"], sum(n), 8)
        if zero is not None:
            starts[2::41] = zero[1]
        pl = oracle.Plan(rho=0.3, proposal=1) if zero is not None else oracle.Plan(rho=0.3, rjs_cap=64)
        strategy = oracle.AUTO if zero is not None else oracle.RJS_ONLY
        st = torch.from_numpy(starts).to(DEV)
        paths = torch.full((n[0] * 10 + n[1] * 7,), -7, dtype=torch.int32, device=DEV)
        lengths = torch.full((sum(n),), -7, dtype=torch.int32, device=DEV)
        lg = fw_logic(N2V)
        qs = [fw.fw_query(lg, n[0], L[0], 70, 0, 0, 0), fw.fw_query(lg, n[1], L[1], 71, n[0], n[0] * 10, n[0])]
        b = fw.fw_batch_create(gg.handle, qs, fw_plan(pl), strategy, st, paths, lengths)
        s = torch.cuda.Stream()
        fw.fw_batch_capture(b, None, s)
        for replay in (False, True, True):
            paths.fill_(-7)
            lengths.fill_(-7)
            torch.cuda.synchronize()
            if replay:
                fw.fw_batch_replay(b, s)
            else:
                fw.fw_batch_launch(b)
            torch.cuda.synchronize()
            for q0, o, w, i in ((0, 0, 10, 0), (5, 50, 7, 1)):
                p, ln, _ = gpu_walk(gg, N2V, pl, strategy, starts[q0:q0 + n[i]], L[i], 70 + i)
                np.testing.assert_array_equal(paths[o:o + n[i] * w].view(n[i], w).cpu().numpy(), p)
                np.testing.assert_array_equal(lengths[q0:q0 + n[i]].cpu().numpy(), ln)
        fw.fw_batch_destroy(b)
    finally:
        gg.close()

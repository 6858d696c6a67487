"""The forms a walk launch takes (needs an MI355X): launches large enough to leave the eRVS scan
out of the kernel, whose walks that do meet an eRVS step are parked and run on by a second
launch, and the 64-byte parts in which paths are written.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests._gpu import GpuGraph, assert_parity, fw_logic, fw_plan, gpu_walk, parity
from tests.test_gpu_parity import N2V, MP

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
PR2 = oracle.Logic(kind=oracle.SECOND_PR, weighted=True, gamma=0.2)
N = (1 << 18) + 777  # more walkers than the form with the scan has lanes
DEV = torch.device("cuda:0")


def _graph(heavy: bool):
    """Scale 9: `heavy` gives a few edges 10^4 times the weight (trials run into the cap), else
    the edges at every eighth vertex weigh 0 (such rows go to eRVS under h-proportional proposals)."""
    g = synth.rmat(9, 8 << 9, seed=4, nlabels=5)
    src = np.repeat(np.arange(g["nv"]), np.diff(g["row_ptr"]))
    lo, hi = np.minimum(src, g["col"]), np.maximum(src, g["col"])
    if heavy:
        g["h"] = np.where((lo * 31 + hi * 17) % 97 == 0, g["h"] * np.float32(1e4), g["h"]).astype(np.float32)
    else:
        g["h"] = np.where((lo % 8 == 0) | (hi % 8 == 0), np.float32(0), g["h"])
    return g


@pytest.mark.parametrize("logic", ["node2vec", "secondpr", "metapath"])
@pytest.mark.parametrize("case", ["cap", "zero_rows"])
def test_parked_walks(logic, case):
    """Counter-free launches (scan-free form, parked walks resumed) equal counted ones (scan in
    the kernel) on every walker, and the oracle on the first 3000."""
    print("parked", logic, case, flush=True)
    g = _graph(case == "cap")
    lg = {"node2vec": N2V, "secondpr": PR2, "metapath": MP}[logic]
    gg = GpuGraph(g, index=True, alias=True)
    try:
        starts = synth.uniform_starts(g["nv"], N, 9)
        if case == "cap":
            pl, strategy = oracle.Plan(rho=0.3, rjs_cap=64), oracle.RJS_ONLY
        else:
            pl, strategy = oracle.Plan(rho=0.3, proposal=1), oracle.AUTO
        p0, l0, st = gpu_walk(gg, lg, pl, strategy, starts, 7, 3)
        p1, l1, _ = gpu_walk(gg, lg, pl, strategy, starts, 7, 3, counters=False)
        assert case != "cap" or st["rjs_fallbacks"] > 1000
        np.testing.assert_array_equal(p1, p0)
        np.testing.assert_array_equal(l1, l0)
        ora = oracle.walk(oracle.Graph(g), lg, pl, strategy, starts[:3000], 7, 3)
        assert_parity(parity(p1[:3000], l1[:3000], ora))
    finally:
        gg.close()


def test_parked_walks_of_a_batch():
    """A batch of two queries past the same size, with zero rows: each equals its own fw_walk."""
    g = _graph(False)
    gg = GpuGraph(g, index=True, alias=True)
    try:
        n = np.array([5, N], np.int64)
        L = [9, 6]
        starts = torch.from_numpy(synth.uniform_starts(g["nv"], int(n.sum()), 8)).to(DEV)
        paths = torch.full((int(5 * 10 + N * 7),), -7, dtype=torch.int32, device=DEV)
        lengths = torch.full((int(n.sum()),), -7, dtype=torch.int32, device=DEV)
        plan = fw_plan(oracle.Plan(rho=0.3, proposal=1))
        lg = fw_logic(N2V)
        qs = [fw.fw_query(lg, 5, 9, 70, 0, 0, 0), fw.fw_query(lg, N, 6, 71, 5, 50, 5)]
        b = fw.fw_batch_create(gg.handle, qs, plan, fw.FW_AUTO, starts, paths, lengths)
        for _ in range(2):
            fw.fw_batch_launch(b)
        torch.cuda.synchronize()
        for i, (q0, o, w) in enumerate(((0, 0, 10), (5, 50, 7))):
            k = int(n[i])
            p, ln, _ = gpu_walk(gg, N2V, oracle.Plan(rho=0.3, proposal=1), oracle.AUTO,
                                starts[q0:q0 + k].cpu().numpy(), L[i], 70 + i)
            np.testing.assert_array_equal(paths[o:o + k * w].view(k, w).cpu().numpy(), p)
            np.testing.assert_array_equal(lengths[q0:q0 + k].cpu().numpy(), ln)
        fw.fw_batch_destroy(b)
    finally:
        gg.close()


@pytest.mark.parametrize("L", [0, 1, 2, 14, 15, 16, 17, 31, 48, 130])
def test_path_parts_at_every_alignment(L):
    """Paths starting at each of the 16 places of a 64-byte part, some walks ending early: only
    the rows themselves are written."""
    g = synth.rmat(8, 2 << 8, seed=6)  # sparse: dead ends and isolated vertices
    gg = GpuGraph(g, index=True, alias=True)
    try:
        n = 61
        starts = synth.uniform_starts(g["nv"], n, 2)
        st = torch.from_numpy(starts).to(DEV)
        pl = oracle.Plan(rho=0.3, proposal=1, bound=2)
        ora = oracle.walk(oracle.Graph(g), N2V, pl, oracle.AUTO, starts, L, 5)
        for off in range(16):
            print("parts", L, off, flush=True)
            buf = torch.full((n * (L + 1) + 64,), -9, dtype=torch.int32, device=DEV)
            lengths = torch.full((n,), -7, dtype=torch.int32, device=DEV)
            fw.fw_walk(gg.handle, fw_logic(N2V), fw_plan(pl), fw.FW_AUTO, st, n, L, 5, buf[16 + off:], lengths)
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert (got[:16 + off] == -9).all() and (got[16 + off + n * (L + 1):] == -9).all()
            p = got[16 + off:16 + off + n * (L + 1)].reshape(n, L + 1)
            assert_parity(parity(p, lengths.cpu().numpy(), ora) if L else
                          {"unflagged": [] if (p[:, 0] == starts).all() else ["start"], "flagged": [], "steps": 1})
    finally:
        gg.close()


def test_served_results_with_and_without_pinned_room():
    """Results and starts that find room in the server's 32 MiB of pinned memory and those that do
    not (nothing is fetched before all are done): odd sizes, single walkers, paths of one slot."""
    g = _graph(False)
    gg = GpuGraph(g, alias=True, index=True)
    pl = oracle.Plan(rho=1.0, proposal=1)
    rng = np.random.default_rng(11)
    jobs = [(int(n), int(L), 50 + i) for i, (n, L) in enumerate(
        [(1, 1), (3, 0), (60001, 40), (1, 100), (70003, 39), (5, 7), (90001, 31), (0, 5), (64, 3), (80000, 33), (2, 2)])]
    try:
        srv = fw.fw_server_create(gg.handle, fw_plan(pl), fw.FW_AUTO, 1 << 28, 16, 8, 64)
        try:
            sent = {}
            for n, L, seed in jobs:
                st = rng.integers(0, g["nv"], n).astype(np.int32)
                sent[fw.fw_server_submit(srv, fw_logic(N2V), st, L, seed)] = (st, n, L, seed)
            left = set(sent)
            while left:
                left.discard(fw.fw_server_next_done(srv, 1000))
            got = {i: fw.fw_server_result(srv, i, n, L)[:2] for i, (st, n, L, seed) in sent.items()}
        finally:
            fw.fw_server_destroy(srv)
        for i, (st, n, L, seed) in sent.items():
            p, ln, _ = gpu_walk(gg, N2V, pl, oracle.AUTO, st, L, seed, counters=False)
            np.testing.assert_array_equal(got[i][0].reshape(n, L + 1), p)
            np.testing.assert_array_equal(got[i][1], ln)
    finally:
        gg.close()

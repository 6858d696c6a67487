"""What fw_plan_autotune keeps at its default (needs an MI355X): fields that cannot change the
sample walks' launches must not be chosen by the noise of timing them.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from tests._gpu import GpuGraph

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _rvs_steps(gg, logics, plan):
    """eRVS steps that the plan takes on walks as the tuner samples them."""
    n, L = min(gg.nv, 1 << 18), 16
    starts = torch.from_numpy(synth.uniform_starts(gg.nv, n, 1)).to(DEV)
    paths = torch.empty((n, L + 1), dtype=torch.int32, device=DEV)
    lengths = torch.empty(n, dtype=torch.int32, device=DEV)
    stats = torch.zeros(fw.FW_NSTATS, dtype=torch.int64, device=DEV)
    for lg in logics:
        fw.fw_walk(gg.handle, lg, plan, fw.FW_AUTO, starts, n, L, 3, paths, lengths, stats)
    torch.cuda.synchronize()
    st = dict(zip(fw.STAT_NAMES, stats.tolist()))
    return st["rvs_steps"] + st["rjs_fallbacks"]


@pytest.mark.parametrize("scale", [12, 19])
@pytest.mark.parametrize("logic", ["node2vec", "metapath", "mix"])
def test_tuned_plan_without_ervs_keeps_defaults(scale, logic):
    """Twelve tunings: a plan whose sampled steps are all eRJS keeps the default lds_cap, lanes and
    thresholds (kernels of both sizes: with the scan compiled in, and without)."""
    print("autotune", scale, logic, flush=True)
    mp = logic == "metapath"
    g = synth.rmat(scale, 8 << scale, seed=3, nlabels=5 if mp else 0)
    gg = GpuGraph(g, index=True, alias=True, label_alias=mp)
    try:
        d = fw.fw_plan_default()
        n2v = [fw.fw_logic_node2vec(0.5, 2.0, True), fw.fw_logic_node2vec(1.0, 2.0, True)]
        logics = [fw.fw_logic_metapath([0, 1, 2, 3, 4], True)] if mp else n2v[:1] if logic == "node2vec" else n2v
        without = 0
        for _ in range(12):
            pl = fw.fw_plan_autotune_mix(gg.handle, logics)
            # (rho below 1/2 sends every step of these logics to eRJS by the cost model)
            if pl.rho >= 0.5 or pl.d_lo > 1 or pl.rjs_cap < 64 or _rvs_steps(gg, logics, pl) > 0:
                continue
            without += 1
            assert (pl.lds_cap, pl.hub_deg, pl.hub_lanes, pl.rvs_share) == (d.lds_cap, d.hub_deg, d.hub_lanes, d.rvs_share)
        print("tunings without eRVS:", without, flush=True)
    finally:
        gg.close()

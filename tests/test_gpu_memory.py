"""Device memory after graphs are destroyed (needs an MI355X)."""
from __future__ import annotations

import pytest
import torch

import synth
from tests._gpu import GpuGraph

import paper_2512_00705_amd as fw

pytestmark = pytest.mark.gpu


def test_memory_goes_back():
    """A first graph's memory goes back when it is destroyed; that of graphs made one after another is
    kept until fw_memory_release."""
    g = synth.rmat(16, 16 << 16, seed=2)
    of_graph = 64 * g["ne"]  # the proposal records alone

    def taken(free0):
        torch.cuda.synchronize()
        return free0 - torch.cuda.mem_get_info()[0]

    GpuGraph(synth.rmat(8, 8 << 8, seed=2), index=True, alias=True).close()  # (what a process's first kernels take)
    fw.fw_memory_release()
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    for kept in (False, True, True):
        gg = GpuGraph(g, index=True, alias=True)
        torch.cuda.empty_cache()
        assert taken(free0) > of_graph
        gg.close()
        gg.t = None
        torch.cuda.empty_cache()
        print("kept", kept, taken(free0), of_graph, flush=True)
        assert (taken(free0) > of_graph) if kept else (taken(free0) < of_graph // 4), (kept, taken(free0))
    fw.fw_memory_release()
    assert taken(free0) < of_graph // 4

"""What the compiler gives the kernels that sample by eRVS (CPU: a compile for gfx950).

A weight chosen through a reference became a load of a chosen address, with the step's weights in
scratch memory: every edge of a scan waited for it.  The forms without counters must need none.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from tests.conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_2512_00705_amd", "csrc")


def _resources(source, tmp_path):
    """{mangled kernel name: {"VGPRs": .., "ScratchSize": .., ...}} of one source."""
    import importlib.util

    spec = importlib.util.spec_from_file_location("_fw_build", os.path.join(ROOT, "paper_2512_00705_amd", "_build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    r = subprocess.run([HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, source), "-o",
                        str(tmp_path / "k.s"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: (?:.*: )?\s*([A-Za-z ]+?)(?: \[[^\]]*\])?: (\S+)", line)
        if not m:
            continue
        if m.group(1) == "Function Name":
            cur = out.setdefault(m.group(2), {})
        elif cur is not None and m.group(2).isdigit():
            cur[m.group(1)] = int(m.group(2))
    return out


@pytest.mark.skipif(not shutil.which(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,forms", [
    ("fw_rvs.hip", r"rvs_kernelILi\dELb\dELb0ELi1E"),                          # no counters, no hub lanes
    ("fw_trial_node2vec.hip", r"walk_kernelILi\dELb\dELi\dELb\dELb0ELi[01]E"),  # no counters, no hub lanes
])
def test_no_scratch_memory(source, forms, tmp_path):
    res = {k: v for k, v in _resources(source, tmp_path).items() if re.search(forms, k)}
    assert len(res) >= 6, sorted(res)
    for name, r in res.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        assert r["Occupancy"] >= (7 if source == "fw_rvs.hip" else 4), (name, r)

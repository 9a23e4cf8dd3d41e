"""The systems of test_gpu_step_merged.py take the path that it compares: the force
pass with the finalize as one of its blocks up to 512 step-pass blocks, the two
launches above, seen in the kernels that a step launches (torch's profiler, in a
process of its own); and their lists are rebuilt on the way."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CASES = [("lj", 30, 4, 0, 0, True), ("lj", 257, 7, 0, 0, True), ("lj", 1021, 8, 1, 0, True),
         ("lj", 1100, 16, 1, 1, True), ("lj", 2048, 64, 0, 0, True), ("lj", 2052, 64, 0, 1, False),
         ("water", 387, 8, 0, 0, True), ("water", 1536, 33, 1, 1, True)]
CHILD = r"""
import json, sys
sys.path.insert(0, %(root)r)
import torch
from torch.profiler import ProfilerActivity, profile
from paper_2602_13553_amd import inputs, pimd
for kind, N, P, fixcom, obabo, merged in %(cases)r:
    spec = (inputs.lj_liquid if kind == "lj" else inputs.water)(n_atoms=N, n_beads=P, seed=N)
    spec.fixcom = fixcom
    spec.integrator = pimd.PIMD_OBABO if obabo else pimd.PIMD_BAOAB
    spec.skin = 0.05 if kind == "lj" else spec.skin
    ctx = pimd.Context.from_spec(spec, flags=pimd.PIMD_FLAG_VALU_TRANSFORMS)
    out = {"blocks": ctx.launch_info()["fused_blocks"]}
    ctx.set_state(spec.x0, spec.v0, 0)
    ctx.step(70)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        ctx.step(4)
        torch.cuda.synchronize()
    out["rebuilds"] = ctx.estimators()["n_rebuilds"]
    ctx.close()
    for k in ("k_pair_step<", "k_pair<", "k_fused<0"):
        out[k] = sum(e.count for e in prof.key_averages() if k in e.key)
    print("CASE " + json.dumps(out), flush=True)
"""


def test_step_routes():
    r = subprocess.run([sys.executable, "-c", CHILD % {"root": ROOT, "cases": CASES}], capture_output=True,
                       text=True, timeout=100)
    print(r.stdout[-3000:], flush=True)
    assert r.returncode == 0, r.stderr[-3000:]
    got = [json.loads(line[5:]) for line in r.stdout.splitlines() if line.startswith("CASE ")]
    assert len(got) == len(CASES)
    for (kind, N, P, _, _, merged), g in zip(CASES, got):
        assert (g["blocks"] <= 512) == merged, (kind, N, P, g)
        assert g["k_fused<0"] == 4, (kind, N, P, g)
        assert g["k_pair_step<"] == (4 if merged else 0), (kind, N, P, g)
        assert g["k_pair<"] == (0 if merged else 4), (kind, N, P, g)
        assert g["rebuilds"] > 1, (kind, N, P, g)

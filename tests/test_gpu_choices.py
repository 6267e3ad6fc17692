"""Which of a setup's ways each kind of plan takes (the FMM_LOG line "choices"):
the M2L kernel's workgroups a CU, the evaluation's waves an item. The accuracy on each of them is tested
elsewhere; here a changed rule or kernel that no longer reaches one shows."""

import json
import os
import re
import subprocess
import sys

import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PLANS = {
    "few_big_leaves": dict(shape="cube", n=200_576, order=7, basis=1, precision=2, leaf=400),
    "many_short_items": dict(shape="line", n=267_667, order=6, basis=1, precision=1, nrhs=3, outputs=2, leaf=16),
    "few_points": dict(shape="cube", n=100, order=4, leaf=64),
    "order10": dict(shape="cube", n=3000, order=10, eps=1e-8, leaf=64),
}

SCRIPT = """
import json, sys
import numpy as np
import torch
import paper_1605_01715_amd as F
import workloads as W
for name, c in json.loads(sys.argv[1]).items():
    n, rng = c["n"], np.random.default_rng(c["n"])
    if c["shape"] == "sphere":
        x = rng.standard_normal((n, 3))
        x /= np.linalg.norm(x, axis=1, keepdims=True)
    elif c["shape"] == "cloud":
        x = W.clustered(n, seed=1)["xyz"]
    elif c["shape"] == "line":
        t = rng.random(n)
        x = np.stack([t, t * t, 0.3 + 0.1 * t], 1)
    else:
        x = rng.random((n, 3))
    o = F.fmm_default_options(order=c["order"], basis=c.get("basis", 0), leaf_size=c["leaf"], pinv_eps=c.get("eps", 0.0),
                              precision=c.get("precision", 0), nrhs=c.get("nrhs", 1), outputs=c.get("outputs", 1),
                              uniform_depth=c.get("depth", 0))
    sys.stderr.write("plan " + name + "\\n")
    sys.stderr.flush()
    F.fmm_destroy(F.fmm_setup(torch.from_numpy(np.ascontiguousarray(x, np.float32)).to("cuda:0"), options=o))
"""


@pytest.fixture(scope="module")
def choices():
    say("test_gpu_choices: " + ", ".join(PLANS))
    out = subprocess.run([sys.executable, "-c", SCRIPT, json.dumps(PLANS)], cwd=ROOT, timeout=100, text=True,
                         capture_output=True, env=dict(os.environ, FMM_LOG="1"))
    assert out.returncode == 0, out.stderr[-2000:]
    got, name = {}, None
    for line in out.stderr.splitlines():
        if line.startswith("plan "):
            name = line[5:]
        if "choices:" in line:
            got[name] = {k: float(v) for k, v in re.findall(r"(\w+)=([-\d.]+)", line)}
    for name, c in got.items():
        say(f"  {name}: {c}")
    return got


def test_two_workgroups_a_cu_at_256_rows(choices):
    assert choices["order10"]["rows"] == 256 and choices["order10"]["blocks"] >= 2


def test_evaluation_waves(choices):
    assert choices["few_big_leaves"]["eval_waves"] >= 4  # 3.5 items for each SIMD
    assert choices["many_short_items"]["eval_waves"] == 1
    assert choices["few_points"]["eval_waves"] == 1

"""Which of a setup's ways each kind of plan takes (the FMM_LOG line "choices"):
the M2L kernel and its workgroups a CU, the line below which its tiles are
regrouped and the directions that share a tile, the evaluation's waves an item
and whether it starts beside the M2L kernel or after it. The accuracy on each of
them is tested elsewhere; here a changed rule or kernel that no longer reaches
one shows."""

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
    "sheet": dict(shape="sphere", n=100_000, order=6, basis=1, nrhs=2, leaf=64),
    "sheet_bf16x3": dict(shape="sphere", n=100_000, order=6, basis=1, nrhs=2, leaf=64, precision=2),
    "cloud": dict(shape="cloud", n=300_000, order=6, leaf=64),
    "sheet_o5": dict(shape="sphere", n=60_000, order=5, basis=1, leaf=64),
    "small_sheet": dict(shape="sphere", n=3000, order=6, leaf=16),
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


def test_evaluation_beside_or_after_the_translation(choices):
    assert choices["sheet"]["eval_after"] == 1         # many even tiles, float32
    assert choices["sheet_bf16x3"]["eval_after"] == 0  # waits on memory
    assert choices["cloud"]["eval_after"] == 0         # the longest piece is all of it
    assert choices["sheet_o5"]["lean"] == 1            # the longest piece is less than the rest,
    assert choices["sheet_o5"]["eval_after"] == 0      # but more than half of it


def test_tiles_and_kernel_of_the_translation(choices):
    assert choices["cloud"]["fill"] == 0.65 and choices["sheet_bf16x3"]["fill"] == 0.45
    assert choices["cloud"]["pair_tiles"] > 0 and choices["cloud"]["group"] > 1 and choices["sheet"]["group"] > 1
    assert choices["small_sheet"]["pair_tiles"] > 0 and choices["small_sheet"]["group"] == 1  # fewer tiles than slots
    assert choices["sheet"]["lean"] == 1 and choices["sheet"]["blocks"] == 3 and choices["cloud"]["lean"] == 0

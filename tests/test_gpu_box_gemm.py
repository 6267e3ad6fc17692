"""The float64 box GEMM with one, two, four and eight waves per output block:
the surface form on trees of more and more boxes (its M2M, L2L, projections
and expansions all run on it), against the direct sum.

Order 6 in float32 reaches a few 1e-6 on uniform points; a wrong, dropped or
doubled partial sum shows as an error of order 1e-2 or more."""

import numpy as np
import pytest

import workloads as W
from oracle import direct as D

from gpu_common import errors, fmm_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(700, 64), (6000, 24), (12000, 12), (16000, 6), (24000, 3)])
@pytest.mark.parametrize("order", [6, 8])
def test_split_box_gemms(n, leaf, order):
    d = W.cube_uniform(n, seed=n)
    x, q = d["xyz"], d["q"]
    nrhs = 2 if n <= 6000 else 1
    qq = np.stack([q, q[::-1]])[:nrhs]
    r = fmm_run(x, q=qq, order=order, leaf=leaf, root=d["root"], nrhs=nrhs)
    say(f"test_split_box_gemms: n={n} leaf={leaf} order={order} boxes={r['info']['n_boxes']} rank={r['info']['rank']}")
    for k in range(nrhs):
        ref, _ = D.direct_sum(x, x, qq[k])
        l2, worst = errors(r["pot"][k], ref)
        say(f"  rel L2 {l2:.2e}, worst {worst:.2e}")
        assert l2 < 2e-5 and worst < 2e-3

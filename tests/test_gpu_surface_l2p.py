"""The surface form's L2P, which stages a leaf's whole downward surface (one to
five tiles of 64 points): 1 to 100 targets a leaf, the potential and the field,
one to four right-hand sides, against the direct sum.

The form's error on uniform points is about 1e-4, 3e-6 and 5e-7 at orders 4, 6
and 8 (the field's up to ten times that); a tile left out, read twice or mixed
with the next one's records shows as 1e-2 or more."""

import numpy as np
import pytest

import workloads as W
from oracle import direct as D

from gpu_common import errors, fmm_run, say

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 3, 7, 15, 21, 22, 31, 32, 33, 43, 45, 63, 64, 65, 100, 0]


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("order,nrhs,bound", [(4, 1, 1e-3), (6, 1, 5e-5), (6, 4, 5e-5), (7, 3, 2e-5), (8, 1, 1e-5),
                                              (8, 2, 1e-5)])
def test_l2p_over_targets_per_leaf(order, nrhs, bound, field):
    d = W.cube_uniform(4000, seed=order)
    x = d["xyz"]
    rng = np.random.default_rng(order)
    q = rng.standard_normal((nrhs, len(x))).astype(np.float32)
    lo, side = x.min(0), (x.max(0) - x.min(0)) / 4
    cells = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3)
    t = np.concatenate([lo + side * (c + 0.02 + 0.96 * rng.random((COUNTS[i % len(COUNTS)], 3)))
                        for i, c in enumerate(cells)]).astype(np.float32)
    r = fmm_run(x, q=q, trg=t, field=field, order=order, depth=2, root=d["root"], nrhs=nrhs)
    say(f"test_l2p_over_targets_per_leaf: order={order} nrhs={nrhs} field={field} targets={len(t)}")
    for k in range(nrhs):
        pot, fld = D.direct_sum(t, x, q[k], potential=not field, field=field)
        l2, worst = errors(r["field"][k], fld) if field else errors(r["pot"][k], pot)
        say(f"  rel L2 {l2:.2e}, worst {worst:.2e}")
        b = 10 * bound if field else bound
        assert l2 < b and worst < 100 * b

"""The Chebyshev L2P of 8 nodes a side, which takes 16 targets at a time: 1 to
100 targets a leaf (items of 64 and a remainder), the potential and the field,
one to four right-hand sides, against the direct sum.

The form's error at 8 nodes per axis is about 1e-6 (the field's about 1e-5); a
target that took another's weights, or a wrong half of the nodes, shows as 1e-2
or more."""

import numpy as np
import pytest

import workloads as W
from oracle import direct as D

from gpu_common import errors, fmm_run, say

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 81, 100, 0]


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4])
def test_l2p_over_targets_per_leaf(nrhs, field):
    d = W.cube_uniform(4000, seed=nrhs)
    x = d["xyz"]
    rng = np.random.default_rng(nrhs)
    q = rng.standard_normal((nrhs, len(x))).astype(np.float32)
    lo, side = x.min(0), (x.max(0) - x.min(0)) / 4
    cells = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3)
    t = np.concatenate([lo + side * (c + 0.02 + 0.96 * rng.random((COUNTS[i % len(COUNTS)], 3)))
                        for i, c in enumerate(cells)]).astype(np.float32)
    r = fmm_run(x, q=q, trg=t, field=field, order=8, depth=2, root=d["root"], nrhs=nrhs, basis=1)
    say(f"test_l2p_over_targets_per_leaf: nrhs={nrhs} field={field} targets={len(t)} leaves={r['info']['n_leaves']}")
    for k in range(nrhs):
        pot, fld = D.direct_sum(t, x, q[k], potential=not field, field=field)
        l2, worst = errors(r["field"][k], fld) if field else errors(r["pot"][k], pot)
        say(f"  rel L2 {l2:.2e}, worst {worst:.2e}")
        assert l2 < (2e-4 if field else 2e-5) and worst < (2e-2 if field else 2e-3)

"""The Chebyshev form over the numbers of boxes at which its kernels change:
P2M with four waves a leaf below 1024 leaves, the basis changes with eight,
four, two waves or one workgroup per 32 rows as the boxes grow, M2M with a
missing child; against the direct sum.

The form's error at 8, 7 and 5 nodes per axis is about 1e-6, 1e-5 and 1e-4 here;
a wrong, dropped or doubled part shows as 1e-2 or more."""

import numpy as np
import pytest

import workloads as W
from oracle import direct as D

from gpu_common import errors, fmm_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(150, 16), (3000, 48), (9000, 24), (14_000, 8), (20_000, 4)])
@pytest.mark.parametrize("order,nrhs,bound", [(8, 1, 2e-5), (7, 3, 1e-4), (5, 2, 2e-3)])
def test_chebyshev_over_box_counts(n, leaf, order, nrhs, bound):
    d = W.clustered(n, seed=n, n_blobs=4)
    x, nrm = d["xyz"], d["normals"]
    rng = np.random.default_rng(n)
    q, mu = (rng.standard_normal((nrhs, n)).astype(np.float32) for _ in range(2))
    mu *= 0.02  # dipoles of about the leaf size: both layers count
    r = fmm_run(x, q=q, mu=mu, nrm=nrm, order=order, leaf=leaf, root=d["root"], nrhs=nrhs, basis=1)
    say(f"test_chebyshev_over_box_counts: n={n} leaf={leaf} order={order} boxes={r['info']['n_boxes']} "
        f"leaves={r['info']['n_leaves']}")
    for k in range(nrhs):
        ref, _ = D.direct_sum(x, x, q[k], mu[k][:, None].astype(np.float64) * nrm)
        l2, worst = errors(r["pot"][k], ref)
        say(f"  rel L2 {l2:.2e}, worst {worst:.2e}")
        assert l2 < bound and worst < 100 * bound

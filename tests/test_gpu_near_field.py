"""The leaf evaluation alone (a tree of one level: every pair is a near pair)
where one, two, four or eight waves share a work item's sources, against the
oracle's float64 direct sum.

A few leaves with n sources each give items of n / 64 source tiles, shared by
the fewest waves that keep two tiles each: 1 wave below 256 sources, 8 from
about 1024. The sizes straddle those and leave partial tiles and ranges. A
term is off by at most about 16 roundings and a float32 partial sum of one
tile by 64 more: 80 * 2^-24 of the sum of the terms' magnitudes."""

import numpy as np
import pytest

from oracle import direct as D

from gpu_common import fmm_run, say

pytestmark = pytest.mark.gpu

BOUND = 80 * 2.0 ** -24


@pytest.mark.parametrize("n", [9, 130, 257, 521, 1030, 2500])
@pytest.mark.parametrize("layers,field,nrhs", [("s", False, 1), ("d", False, 1), ("sd", False, 1), ("s", True, 1),
                                               ("d", False, 3), ("sd", False, 4), ("s", True, 2)])
def test_items_shared_by_waves(n, layers, field, nrhs):
    say(f"test_items_shared_by_waves: n={n} layers={layers} field={field} nrhs={nrhs}")
    rng = np.random.default_rng(n + nrhs)
    x = (rng.random((n, 3)) ** 2).astype(np.float32)  # uneven leaves
    x[n // 2] = x[0]                                   # a coincident pair is left out
    nrm = rng.standard_normal((n, 3)).astype(np.float32) if "d" in layers else None
    q = rng.standard_normal((nrhs, n)).astype(np.float32) if "s" in layers else None
    mu = rng.standard_normal((nrhs, n)).astype(np.float32) if "d" in layers else None
    got = fmm_run(x, q=q, mu=mu, nrm=nrm, field=field, depth=1, root=(0.0, 0.0, 0.0, 1.0), nrhs=nrhs)
    d = x[:, None].astype(np.float64) - x[None].astype(np.float64)
    r = np.linalg.norm(d, axis=2)
    inv = np.where(r < 1e-5, 0.0, 1.0 / np.where(r == 0, 1.0, r))
    for k in range(nrhs):
        dip = (mu[k][:, None] * nrm) if mu is not None else None
        pot, fld = D.direct_sum(x, x, q[k] if q is not None else None, dip, potential=not field, field=field)
        mag = np.zeros(n)
        if q is not None:
            mag += (inv ** (2 if field else 1)) @ np.abs(q[k])
        if dip is not None:
            mag += inv ** 2 @ np.linalg.norm(dip, axis=1)
        err = np.linalg.norm(got["field"][k] - fld, axis=1) / np.sqrt(3.0) if field else np.abs(got["pot"][k] - pot)
        assert np.all(err <= BOUND * mag / (4 * np.pi) + 1e-30), (k, err.max())

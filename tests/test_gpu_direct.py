"""The all-pairs kernel at the edges of its work split (targets per workgroup,
slices, tiles of 1024 sources) against the oracle's float64 direct sum.

A term is off by at most about 16 roundings and a float32 partial sum of at
most 64 terms by 64 more, so a target's error is within 80 * 2^-24 of the sum
of the magnitudes of its terms."""

import numpy as np
import pytest

from oracle import direct as D

from gpu_common import dev, say

pytestmark = pytest.mark.gpu

BOUND = 80 * 2.0 ** -24


def _magnitudes(trg, src, q, dip, field):
    d = trg[:, None].astype(np.float64) - src[None].astype(np.float64)
    r = np.linalg.norm(d, axis=2)
    inv = np.where(r < 1e-5, 0.0, 1.0 / np.where(r == 0, 1.0, r))
    if field:
        return (inv ** 2 @ np.abs(q)) / (4 * np.pi)
    m = inv @ np.abs(q) if q is not None else 0.0
    if dip is not None:
        m = m + (inv ** 2) @ np.linalg.norm(dip, axis=1)
    return m / (4 * np.pi)


@pytest.mark.parametrize("n_trg,n_src", [(1, 1), (1, 2050), (3, 1024), (255, 1025), (257, 33), (801, 801),
                                         (1025, 1023), (2049, 4097), (4099, 3000), (20000, 65)])
@pytest.mark.parametrize("layers,out", [("s", "pot"), ("d", "pot"), ("sd", "pot"), ("s", "field"), ("s", "both")])
def test_direct_at_the_edges_of_its_split(n_trg, n_src, layers, out):
    import torch

    import paper_1605_01715_amd as F

    say(f"test_direct_at_the_edges_of_its_split: {n_trg} targets, {n_src} sources, {layers}, {out}")
    rng = np.random.default_rng(n_trg + 7 * n_src)
    src = rng.random((n_src, 3)).astype(np.float32)
    trg = rng.random((n_trg, 3)).astype(np.float32)
    trg[: min(n_trg, n_src) // 2] = src[: min(n_trg, n_src) // 2]  # coincident pairs are left out
    q = rng.standard_normal(n_src).astype(np.float32) if "s" in layers else None
    nrm = rng.standard_normal((n_src, 3)).astype(np.float32) if "d" in layers else None
    mu = rng.standard_normal(n_src).astype(np.float32) if "d" in layers else None
    pot = torch.full((n_trg,), float("nan"), device="cuda:0") if out != "field" else None
    fld = torch.full((n_trg, 3), float("nan"), device="cuda:0") if out != "pot" else None
    F.fmm_direct(dev(src), dev(trg), q=dev(q) if q is not None else None, mu=dev(mu) if mu is not None else None,
                 src_nrm=dev(nrm) if nrm is not None else None, pot=pot, field=fld)
    torch.cuda.synchronize()
    dip = (mu[:, None] * nrm) if mu is not None else None  # the float32 products the kernel forms
    rp, rf = D.direct_sum(trg, src, q, dip, potential=True, field=out != "pot")
    if pot is not None:
        err = np.abs(pot.cpu().numpy().astype(np.float64) - rp)
        assert np.all(err <= BOUND * _magnitudes(trg, src, q, dip, False) + 1e-30), err.max()
    if fld is not None:
        err = np.linalg.norm(fld.cpu().numpy().astype(np.float64) - rf, axis=1)
        assert np.all(err <= np.sqrt(3.0) * BOUND * _magnitudes(trg, src, q, None, True) + 1e-30), err.max()


def test_direct_non_finite_points():
    """A target that is not finite has no finite potential and spoils no other; a source that is not finite spoils
    every potential; no sources give zeros."""
    import torch

    import paper_1605_01715_amd as F

    rng = np.random.default_rng(0)
    src, q = rng.random((700, 3)).astype(np.float32), rng.standard_normal(700).astype(np.float32)
    for bad in (np.nan, np.inf):
        trg = rng.random((900, 3)).astype(np.float32)
        trg[5, 1] = bad
        pot = torch.zeros(900, device="cuda:0")
        F.fmm_direct(dev(src), dev(trg), q=dev(q), pot=pot)
        fin = np.isfinite(pot.cpu().numpy())
        assert not fin[5] and fin.sum() == 899
        s2 = src.copy()
        s2[699, 2] = bad
        F.fmm_direct(dev(s2), dev(src), q=dev(q), pot=pot[:700])
        assert np.isnan(pot[:700].cpu().numpy()).all()
    F.fmm_direct(dev(src[:0]), dev(src), q=dev(q[:0]), pot=pot[:700])
    assert (pot[:700].cpu().numpy() == 0).all()

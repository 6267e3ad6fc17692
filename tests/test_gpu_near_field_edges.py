"""The leaf evaluation and the L2P at the ends of what they accept: items that
have surfaces and no near points, leaves above level 2, the widest items that
several waves share."""

import numpy as np
import pytest

import test_gpu_near_field as near
from oracle import direct as D

from gpu_common import errors, fmm_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("basis,order,nt", [(0, 6, 64), (0, 6, 200), (1, 6, 64)])
def test_items_with_surfaces_and_no_points(basis, order, nt):
    """Targets in one corner of the root, sources in the opposite one: the
    target leaf has no source beside it, only the far corner's box in its W
    list. The W box holds 4096 points, more than a surface has. Bound: the
    forms' accuracy with a margin; a lost or doubled surface shows as 1e-1."""
    say(f"test_items_with_surfaces_and_no_points: basis={basis} targets={nt}")
    rng = np.random.default_rng(nt)
    trg = (0.05 + 0.1 * rng.random((nt, 3))).astype(np.float32)
    src = (0.8 + 0.15 * rng.random((4096, 3))).astype(np.float32)
    q = rng.random(4096).astype(np.float32)
    got = fmm_run(src, q=q, trg=trg, order=order, leaf=256, root=(0.0, 0.0, 0.0, 1.0), basis=basis)
    assert got["info"]["p2p_pairs"] == 0 and got["info"]["surf_evals"] > 0
    ref, _ = D.direct_sum(trg, src, q)
    l2, worst = errors(got["pot"][0], ref)
    say(f"  rel L2 {l2:.2e}, worst {worst:.2e}")
    assert l2 < 1e-3 and worst < 1e-2


def test_points_closer_than_float32_can_square():
    """A tree of one leaf, all pairs within the tolerance radius: exact zeros,
    also where squared distances to a box surface underflow."""
    say("test_points_closer_than_float32_can_square")
    rng = np.random.default_rng(3)
    x = (1e-24 * rng.random((40, 3))).astype(np.float32)
    q = rng.standard_normal(40).astype(np.float32)
    assert np.array_equal(fmm_run(x, q=q)["pot"][0], np.zeros(40))
    assert np.array_equal(fmm_run(x, q=q, field=True)["field"][0], np.zeros((40, 3)))


def test_target_on_the_surface_of_a_leaf_above_level_two():
    """The root given and a target outside it, where the downward surface of
    the one leaf has a point: every pair is a near pair."""
    say("test_target_on_the_surface_of_a_leaf_above_level_two")
    rng = np.random.default_rng(4)
    src = (2 * rng.random((40, 3)) - 1).astype(np.float32)
    q = rng.standard_normal(40).astype(np.float32)
    trg = np.array([[2.95, 2.95, 2.95], [0.1, 0.2, 0.3]], np.float32)
    got = fmm_run(src, q=q, trg=trg, root=(-1.0, -1.0, -1.0, 2.0))
    pot, _ = D.direct_sum(trg, src, q)
    mag, _ = D.direct_sum(trg, src, np.abs(q))
    assert np.all(np.abs(got["pot"][0] - pot) <= near.BOUND * mag)


@pytest.mark.parametrize("n", [130, 2500])
@pytest.mark.parametrize("nrhs", [3, 4])
def test_field_of_several_densities(n, nrhs):
    """One wave, and eight with up to 128 KB of LDS a workgroup."""
    near.test_items_shared_by_waves(n, "s", True, nrhs)

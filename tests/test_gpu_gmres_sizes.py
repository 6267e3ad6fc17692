"""GMRES where its vectors change their split over blocks (131,072 points) and
the block count ends: the residual that it reports is the one of its solution,
recomputed with fmm_apply (converged or, with few vectors, not)."""

import math

import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu


def _sphere(n):
    import torch

    import paper_1605_01715_amd as F

    g = torch.Generator(device="cuda:0")
    g.manual_seed(n)
    u = torch.randn(n, 3, generator=g, device="cuda:0")
    u = (u / u.norm(dim=1, keepdim=True)).contiguous()
    plan = F.fmm_setup(u, u, options=F.fmm_default_options(order=4, leaf_size=64, basis=1, src_kernels=2))
    w = torch.full((n,), 4 * math.pi / n, device="cuda:0")
    return plan, torch.full((n,), -0.5, device="cuda:0"), w, torch.randn(n, generator=g, device="cuda:0", dtype=torch.float64)


@pytest.mark.parametrize("n,restart", [(65_537, 30), (131_072, 30), (131_073, 5), (524_289, 12)])
def test_residual_at_the_edges_of_the_split(n, restart):
    import torch

    import paper_1605_01715_amd as F

    plan, a, w, b = _sphere(n)
    x = torch.zeros_like(b)
    rc, it, rel = F.gmres_solve(plan, F.FMM_OP_FK, a, None, w, b, x, rtol=1e-5, restart=restart, max_iter=60)
    pot = torch.empty(n, device="cuda:0")
    F.fmm_apply(plan, mu=(x * w.double()).float(), pot=pot)
    r = b - (a.double() * x + pot.double())
    true = float(r.norm() / b.norm())
    say(f"test_residual_at_the_edges_of_the_split: n={n} restart={restart}: {it} iterations, {rel:.3e}, recomputed {true:.3e}")
    assert rc == (F.FMM_OK if rel <= 1e-5 else F.FMM_ERR_NOT_CONVERGED) and rel < 1.0
    assert abs(true - rel) <= 1e-10  # the same float32 products, summed in float64 in another order
    F.fmm_destroy(plan)

"""The all-pairs sum of few sources at many targets (one thread per target,
tiles of 256 sources, sums of at most 64): the edges of its tiles and of the
rule that takes it, against the oracle's float64 direct sum; infinities and NaN;
and that it costs about as much as writing its outputs."""

import numpy as np
import pytest

import test_gpu_direct as base
from gpu_common import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_trg,n_src", [(1, 128), (255, 129), (257, 64), (65536, 1), (65537, 65), (70001, 128),
                                         (70001, 255), (70001, 257), (140000, 513), (70001, 1025), (3, 0)])
@pytest.mark.parametrize("layers,out", [("s", "pot"), ("d", "pot"), ("sd", "pot"), ("s", "field"), ("s", "both")])
def test_few_sources(n_trg, n_src, layers, out):
    base.test_direct_at_the_edges_of_its_split(n_trg, n_src, layers, out)


@pytest.mark.parametrize("n_src", [100, 300])
def test_few_sources_not_finite(n_src):
    import torch

    import paper_1605_01715_amd as F

    say(f"test_few_sources_not_finite: {n_src} sources")
    rng = np.random.default_rng(1)
    src, q = rng.random((n_src, 3)).astype(np.float32), rng.standard_normal(n_src).astype(np.float32)
    trg = rng.random((100_003, 3)).astype(np.float32)
    pot, fld = torch.zeros(len(trg), device="cuda:0"), torch.zeros(len(trg), 3, device="cuda:0")
    for bad in (np.nan, np.inf):
        t2, s2 = trg.copy(), src.copy()
        t2[77, 0] = s2[-1, 2] = bad
        F.fmm_direct(dev(src), dev(t2), q=dev(q), pot=pot, field=fld)
        for out in (pot, fld[:, 0], fld[:, 2]):
            fin = np.isfinite(out.cpu().numpy())
            assert not fin[77] and fin.sum() == len(trg) - 1
        F.fmm_direct(dev(s2), dev(trg), q=dev(q), pot=pot, field=fld)
        assert np.isnan(pot.cpu().numpy()).all() and np.isnan(fld.cpu().numpy()).all()


def test_few_sources_cost_about_their_outputs():
    """1M targets, one source: the launch and 16 MB written. The sliced kernel
    took 67 us for it, seven fills of the same outputs."""
    import torch

    import paper_1605_01715_amd as F

    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    src, q = torch.rand(1, 3, generator=g, device="cuda:0"), torch.rand(1, generator=g, device="cuda:0")
    trg = torch.rand(1_000_000, 3, generator=g, device="cuda:0")
    pot, fld = torch.empty(len(trg), device="cuda:0"), torch.empty(len(trg), 3, device="cuda:0")

    def us(f):
        best = 1e30
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            f()
            a.record()
            for _ in range(20):
                f()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    t_sum = us(lambda: F.fmm_direct(src, trg, q=q, pot=pot, field=fld))
    t_fill = us(lambda: (pot.fill_(1.0), fld.fill_(1.0)))
    say(f"test_few_sources_cost_about_their_outputs: {t_sum:.1f} us, fills {t_fill:.1f}")
    assert t_sum < 3 * t_fill

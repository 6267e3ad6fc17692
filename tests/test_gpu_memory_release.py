"""The memory kept from destroyed plans can be given back, and a plan in use
keeps its own."""

import pytest

import workloads as W

from gpu_common import dev, say

pytestmark = pytest.mark.gpu


def test_kept_memory_is_given_back_on_request():
    import torch

    import paper_1605_01715_amd as F

    say("test_kept_memory_is_given_back_on_request: plans of 300,000 points")
    d = W.clustered(300_000, seed=5)
    x, q = dev(d["xyz"]), dev(d["q"])
    opts = F.fmm_default_options(order=8, leaf_size=64, basis=1, root=d["root"])
    small = F.fmm_setup(x[:3000].contiguous(), options=opts)
    pot, again = torch.empty(3000, device="cuda:0"), torch.empty(3000, device="cuda:0")
    F.fmm_apply(small, q=q[:3000].contiguous(), pot=pot)
    torch.cuda.synchronize()
    F.fmm_release_memory()
    before = torch.cuda.mem_get_info()[0]
    F.fmm_destroy(F.fmm_setup(x, options=opts))
    kept = before - torch.cuda.mem_get_info()[0]
    F.fmm_release_memory()
    left = before - torch.cuda.mem_get_info()[0]
    say(f"  kept {kept >> 20} MB, after the release {left >> 20} MB")
    assert kept > (64 << 20) and left <= (8 << 20)
    F.fmm_apply(small, q=q[:3000].contiguous(), pot=again)
    assert torch.equal(pot, again)
    F.fmm_destroy(small)
    F.fmm_release_memory()

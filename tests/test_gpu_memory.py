"""The memory that plans and solves leave for the next ones: results do not
depend on what a block held before, also with several threads and streams,
and no more than the stated 512 MB stays behind."""

import threading

import numpy as np
import pytest

import workloads as W

from gpu_common import dev, say

pytestmark = pytest.mark.gpu


def _once(d, basis, order, precision, stream=None):
    import torch

    import paper_1605_01715_amd as F

    opts = F.fmm_default_options(order=order, leaf_size=64, src_kernels=3, basis=basis, precision=precision,
                                 root=d["root"])
    plan = F.fmm_setup(d["x"], d["n"], options=opts, stream=stream)
    pot = torch.full((len(d["q"]),), float("nan"), device="cuda:0")
    if stream is not None:
        stream.wait_stream(torch.cuda.default_stream())
    F.fmm_apply(plan, q=d["q"], mu=d["m"], pot=pot, stream=stream)
    F.fmm_destroy(plan)
    torch.cuda.synchronize()
    return pot.cpu().numpy()


def _cloud(n, seed):
    d = W.clustered(n, seed=seed)
    return dict(x=dev(d["xyz"]), n=dev(d["normals"]), q=dev(d["q"]), m=dev(d["mu"]), root=d["root"])


@pytest.mark.parametrize("n", [300, 5000, 40_000])
def test_results_do_not_depend_on_reused_blocks(n):
    say(f"test_results_do_not_depend_on_reused_blocks: n={n}")
    d, other = _cloud(n, 3), _cloud(60_000, 4)
    forms = [(0, 6, 0), (1, 8, 2), (1, 5, 1), (0, 8, 3)]
    first = [_once(d, *f) for f in forms]
    for k, f in enumerate(forms):
        _once(other, *forms[(k + 1) % 4])  # leaves its blocks with other contents
        for _ in range(2):
            assert np.array_equal(_once(d, *f), first[k]), f


def test_threads_and_streams_share_the_kept_blocks():
    import torch

    say("test_threads_and_streams_share_the_kept_blocks: 3 threads, one stream each")
    data = [_cloud(n, 10 + n) for n in (3000, 9000, 20_000)]
    first = [_once(d, 1, 6, 2) for d in data]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        try:
            s = torch.cuda.Stream()
            for i in range(6):
                j = (k + i) % 3
                if not np.array_equal(_once(data[j], 1, 6, 2, stream=s), first[j]):
                    bad.append((k, i))
        except Exception as e:  # reported by the main thread
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


def test_kept_memory_is_bounded():
    import torch

    say("test_kept_memory_is_bounded: plans of up to 400,000 points")
    small = _cloud(300, 1)
    _once(small, 1, 8, 2)
    big = _cloud(400_000, 2)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for _ in range(2):
        _once(big, 1, 8, 2)
    after = torch.cuda.mem_get_info()[0]
    say(f"  kept {(free0 - after) >> 20} MB")
    assert free0 - after <= (512 << 20) + (64 << 20)  # and what torch kept for the outputs
    for _ in range(20):
        _once(small, 1, 8, 2)
    assert free0 - torch.cuda.mem_get_info()[0] <= (64 << 20) + (64 << 20)  # not used again: freed

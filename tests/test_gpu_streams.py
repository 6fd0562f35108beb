"""Builds, products and solves on streams of their own, and from two threads at once:
the arena of a build, the shared pinned pages and the steps queued ahead of their
results are per thread and stream."""
from concurrent.futures import ThreadPoolExecutor
from threading import Barrier

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import say

DEV = "cuda:0"


def work(level, form, stream, turn):
    """Three handles with all their calls, on `stream`; the results on the host."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere
    V, T = icosphere(level)
    out, handles = [], []
    with torch.cuda.stream(stream):
        for seed in range(3):
            turn()
            H = hm.HMatrix(V, T, leaf_size=16 + 8 * seed, eps=1e-6, precision=form)
            handles.append(H)
            g = torch.Generator().manual_seed(seed)
            x = torch.randn((H.n, 5), generator=g, dtype=torch.float64).to(DEV, non_blocking=True)
            out += [H.matvec(x), H.matvec_T(x[:, :1].contiguous())]
            for kw in ({}, {"graph": True}, {"refine": True} if form == "f32" else {"transpose": True}):
                s, info, status = H.solve(x[:, :3].contiguous(), tol=1e-7, **kw)
                assert status == hm.HM_OK
                out += [s, torch.tensor([float(info.iters)], device=DEV)]
        host = [t.cpu() for t in out]
    return handles, host


@pytest.mark.parametrize("levels,forms", [((3, 3), ("f64", "f64")), ((4, 2), ("f32", "f64"))])
def test_two_threads_two_streams(levels, forms):
    """Two threads, each with a stream of its own: the results of one after
    the other on the null stream (every sum has a fixed order: 1e-12)."""
    say("two threads", levels, forms)
    null = torch.cuda.default_stream()
    both = Barrier(2, timeout=60)
    refs = [work(l, f, null, lambda: None) for l, f in zip(levels, forms)]
    with ThreadPoolExecutor(2) as ex:
        runs = [ex.submit(work, l, f, torch.cuda.Stream(), both.wait)
                for l, f in zip(levels, forms)]
        got = [r.result(timeout=100) for r in runs]
    for (_, a), (_, b) in zip(refs, got):
        for u, v in zip(a, b):
            d = (u.double() - v.double()).norm().item()
            assert d <= 1e-12 * u.double().norm().item()
    for handles, _ in refs + got:
        for H in handles:
            H.free()

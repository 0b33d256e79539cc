"""The default plan's choices against what they choose from, by time: a choice
that a rule of sizes makes must not cost what it was made to save.

Bound: the two sides are timed in turn as graph replays, the least of several
rounds each, which repeat to about 2 %; where the rule errs the difference is 15
to 40 %. 1.1 separates the two.
"""
import time

import numpy as np
import pytest
import torch

from paper_2302_00414_amd import workloads as wl

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _graph(call):
    """20 calls in a graph (call keeps its buffers for as long as it lives)."""
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        call()
    s.synchronize()
    with torch.cuda.graph(g, stream=s):
        for _ in range(20):
            call()
    return g


def _times(calls, rounds=8, reps=5):
    """Microseconds per call of every callable, timed in turn."""
    graphs = [_graph(c) for c in calls]
    best = [float("inf")] * len(calls)
    for _ in range(rounds):
        for k, g in enumerate(graphs):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(reps):
                g.replay()
            torch.cuda.synchronize()
            best[k] = min(best[k], (time.perf_counter() - t) / (20 * reps) * 1e6)
    del graphs
    return best


def _nodes(kind, N, M):
    return wl.uniform_nodes(N, 2, 1) if kind == "uniform" else wl.spiral_nodes(N, M)


@pytest.mark.parametrize("prec,kind,M,N,m,nrhs", [
    # few tiles above the density at which many would be the faster way
    ("f64", "spiral", 32, 4096, 2, 1), ("f64", "uniform", 32, 8192, 3, 1),
    ("f64", "uniform", 64, 32768, 4, 1), ("f64", "spiral", 64, 8192, 8, 1),
    ("f64", "spiral", 64, 8192, 4, 11), ("f32", "spiral", 64, 8192, 3, 11),
    ("f64", "uniform", 32, 8192, 6, 2), ("f64", "spiral", 128, 65536, 2, 2),
    # on the other side of the rule's lines
    ("f64", "uniform", 32, 4096, 4, 1), ("f32", "uniform", 32, 400, 4, 1),
    ("f64", "uniform", 256, 120000, 8, 1), ("f32", "uniform", 128, 40321, 6, 11)])
def test_default_spreading_is_not_slower_than_the_lds_kernel(prec, kind, M, N, m, nrhs):
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] {kind} N={N} M={M} m={m} {prec} rhs={nrhs}", flush=True)
    x = _nodes(kind, N, M)
    calls, plans = [], []
    for tuning in (None, {"spread_mode": 1}):
        p = Plan(x, M, 2.0, m, precision=prec, max_rhs=nrhs, tuning=tuning)
        p.set_weights(np.full(N, 1.0 / N))
        v = torch.randn(nrhs, N, dtype=p.cdtype, device="cuda")
        out = torch.empty(nrhs, M * M, dtype=p.cdtype, device="cuda")
        plans.append(p)
        calls.append(lambda p=p, v=v, out=out: p.adjoint(v, out=out))
    default, lds = _times(calls)
    print(f"[time] default {default:.1f} us, LDS kernel {lds:.1f} us", flush=True)
    assert default <= 1.1 * lds
    calls.clear()
    for p in plans:
        p.close()


@pytest.mark.parametrize("prec,M,N,m", [("f64", 128, 76800, 6), ("f64", 256, 1024 * 300, 6),
                                        ("f32", 128, 76800, 6)])
def test_default_items_are_joined_where_that_is_faster(prec, M, N, m):
    """About 300 nodes in every tile: two items each and a sum, or one."""
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] joined N={N} M={M} m={m} {prec}", flush=True)
    x = wl.uniform_nodes(N, 2, 1)
    calls, plans = [], []
    for tuning in (None, {"spread_mode": 7, "item_nodes": 512, "spread_threads": 64}):
        p = Plan(x, M, 2.0, m, precision=prec, tuning=tuning)
        p.set_weights(np.full(N, 1.0 / N))
        v = torch.randn(N, dtype=p.cdtype, device="cuda")
        out = torch.empty(1, M * M, dtype=p.cdtype, device="cuda")
        plans.append(p)
        calls.append(lambda p=p, v=v, out=out: p.adjoint(v, out=out))
    default, joined = _times(calls)
    print(f"[time] default {default:.1f} us, items of 512 {joined:.1f} us", flush=True)
    assert default <= 1.1 * joined
    calls.clear()
    for p in plans:
        p.close()


@pytest.mark.parametrize("kind,M,N,m", [("uniform", 32, 8192, 8), ("uniform", 32, 4096, 6),
                                        ("spiral", 64, 8192, 5)])
def test_forward_of_several_right_hand_sides_fills_the_device(kind, M, N, m):
    """Few work items: five right-hand sides fit beside one another and take
    little longer than one (the grid and its FFT are a few microseconds), where
    one after the other in a work-group they took 1.4 to 1.6 times as long."""
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] forward {kind} N={N} M={M} m={m} f32", flush=True)
    p = Plan(_nodes(kind, N, M), M, 2.0, m, precision="f32", max_rhs=5)
    calls = []
    for nrhs in (1, 5):
        v = torch.randn(nrhs, M * M, dtype=p.cdtype, device="cuda")
        out = torch.empty(nrhs, N, dtype=p.cdtype, device="cuda")
        calls.append(lambda v=v, out=out: p.forward(v, out=out))
    one, five = _times(calls)
    print(f"[time] one {one:.1f} us, five {five:.1f} us", flush=True)
    assert five <= 1.25 * one
    calls.clear()
    p.close()


@pytest.mark.parametrize("d,M,N,m,nrhs,mode", [
    # 3-D: many items of a few nodes at m = 2, m = 1
    (3, 64, 8192, 2, 3, 1), (3, 64, 8192, 2, 1, 1), (3, 32, 60000, 2, 1, 7), (3, 16, 500, 2, 1, 7),
    (3, 64, 8192, 3, 1, 7), (3, 16, 3000, 1, 1, 1),
    # 2-D, few work-groups: by the longest item
    (2, 32, 400, 2, 1, 1), (2, 32, 2400, 2, 1, 7), (2, 32, 400, 3, 1, 7), (2, 32, 2400, 8, 3, 1),
    # many: by the mean item
    (2, 256, 1024 * 100, 2, 1, 1), (2, 256, 1024 * 50, 3, 1, 1), (2, 256, 1024 * 80, 3, 1, 7),
    (2, 256, 1024 * 5, 4, 1, 7)])
def test_float32_default_runs_the_kernel_of(d, M, N, m, nrhs, mode):
    """Each kernel adds in one order of its own: the default plan gives the bits
    of the mode whose kernel the rule takes, and not those of the other."""
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] d={d} N={N} M={M} m={m} f32 rhs={nrhs} -> mode {mode}", flush=True)
    x = wl.uniform_nodes(N, d, 1)
    v = torch.from_numpy(wl.complex_normal((nrhs, N), 2)).to(torch.complex64).cuda()
    out = {}
    for t in (None, 1, 7):
        p = Plan(x, M, 2.0, m, precision="f32", max_rhs=nrhs, tuning=t and {"spread_mode": t})
        p.set_weights(np.full(N, 1.0 / N))
        out[t] = torch.view_as_real(p.adjoint(v))
        p.close()
    other = 8 - mode
    assert torch.equal(out[None], out[mode])
    if m < 8:
        assert not torch.equal(out[None], out[other])

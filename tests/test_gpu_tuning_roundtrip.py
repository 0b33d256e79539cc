"""A plan built from another plan's reported tuning runs the same kernels, and
the autotuner finds the default plan's.

Same kernels give the same bits where a kernel adds in a fixed order (float32,
and the matrix-core kernels in float64); the float64 LDS kernels add with
atomics, so where the default takes them two calls agree to rounding, 1e-14.
"""
import numpy as np
import pytest
import torch

from paper_2302_00414_amd import workloads as wl
from test_gpu_default_choice import _times

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _plan(x, M, m, prec, nrhs, tuning):
    from paper_2302_00414_amd.nfft import Plan
    p = Plan(x, M, 2.0, m, precision=prec, max_rhs=nrhs, tuning=tuning)
    p.set_weights(np.full(x.shape[0], 1.0 / x.shape[0]))
    return p


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("d,M,N,m,nrhs,lds", [
    (2, 32, 4096, 4, 1, False),         # joined items
    (2, 128, 40321, 6, 3, False),
    (2, 128, 256 * 130, 8, 3, False),
    (2, 32, 500, 8, 1, True),
    (3, 16, 3000, 4, 2, False),
    (3, 16, 3000, 1, 1, True)])
def test_a_reported_default_tuning_is_the_default(prec, d, M, N, m, nrhs, lds):
    print(f"[case] d={d} N={N} M={M} m={m} {prec} rhs={nrhs}", flush=True)
    x = wl.uniform_nodes(N, d, 1)
    p = _plan(x, M, m, prec, nrhs, None)
    t = p.tuning()
    q = _plan(x, M, m, prec, nrhs, t)
    assert q.tuning() == t
    from paper_2302_00414_amd.nfft import nfft_footprint
    for k in (p, q):
        assert nfft_footprint(d, M, 2.0, m, N, prec, nrhs) >= k.info()["bytes"]
    v = torch.from_numpy(wl.complex_normal((nrhs, N), 2)).to(p.cdtype).cuda()
    a, b = torch.view_as_real(p.adjoint(v)), torch.view_as_real(q.adjoint(v))
    if lds and prec == "f64":
        assert ((a - b).norm() / a.norm()).item() <= 1e-14
    else:
        assert torch.equal(a, b)
    p.close()
    q.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("M,N,m", [(256, 1024 * 400, 8), (128, 256 * 300, 6)])
def test_autotuned_plan_is_not_slower_than_the_default(prec, M, N, m):
    """At m = 8 only the default mode has the tile kernel, 1.3 to 1.6 times as
    fast here as any other; graph replays timed in turn repeat to about 2 %: 1.1
    separates the two. The winner's reported tuning runs the winner's kernel."""
    print(f"[case] auto N={N} M={M} m={m} {prec}", flush=True)
    x = wl.uniform_nodes(N, 2, 1)
    p, q = _plan(x, M, m, prec, 1, None), _plan(x, M, m, prec, 1, "auto")
    r = _plan(x, M, m, prec, 1, q.tuning())
    v = torch.from_numpy(wl.complex_normal(N, 2)).to(p.cdtype).cuda()
    out = torch.empty(1, M * M, dtype=p.cdtype, device="cuda")
    t = _times([lambda k=k: k.adjoint(v, out=out) for k in (p, q, r)])
    print(f"[time] default {t[0]:.1f}, auto {t[1]:.1f}, again {t[2]:.1f} us {q.tuning()}", flush=True)
    assert t[1] <= 1.1 * t[0] and t[2] <= 1.1 * t[1]
    for k in (p, q, r):
        k.close()


def test_autotuner_times_the_gathers_longest_units_at_speed():
    """32 spiral right-hand sides in one call: units of 768 list entries take
    140 us, of 512 150; timed straight after its plan's making the 768 candidate
    read 147 as the 512 one did, and one plan in five got the slower. Graph
    replays timed in turn repeat to 1 % and the two are 7 % apart: 1.03."""
    M, N = 256, 131072
    x = wl.spiral_nodes(N, M)
    v = torch.from_numpy(wl.complex_normal((32, N), 2)).to(torch.complex64).cuda()
    out = torch.empty(32, M * M, dtype=torch.complex64, device="cuda")
    got = []
    for i in range(8):
        p = _plan(x, M, 6, "f32", 32, "auto")
        got.append(p.tuning())
        p.close()
        print(f"[case] auto spiral, 32 rhs, {i}: {got[-1]}", flush=True)
    best = {"tile_edge": 16, "item_nodes": 768, "fft_min_wg": 64, "spread_mode": 6}
    plans = [_plan(x, M, 6, "f32", 32, t) for t in [best] + [dict(t) for t in {tuple(t.items()) for t in got}]]
    t = _times([lambda k=k: k.adjoint(v, out=out) for k in plans])
    print(f"[time] {[round(k, 1) for k in t]} us", flush=True)
    assert max(t) <= 1.03 * t[0]
    for k in plans:
        k.close()

"""The forward's window sums on the matrix cores (float32; d = 2, m >= 5 and d =
3, m = 4) against the oracle NFFT, at the sizes where the kernel's cuts can go wrong:
groups of 16 nodes that are not full, one node, tiles of several work items,
groups that span more rows than one block of 16 covers, nodes on grid lines
(closed edges) on both axes, a grid of one tile, and right-hand sides that do
not fill the last work-group.

Tolerance: two float32 evaluations of the same transform in different orders
agree to 2e-6, and a float32 transform differs from the oracle by rounding
only: 2e-6 relative l2.
"""
import numpy as np
import pytest
import torch

from oracle import metrics, nfft as onfft
from paper_2302_00414_amd import workloads as wl

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = 2e-6


def _nodes(kind, Ms):
    if kind == "one":
        return np.array([[0.123, -0.4567]])
    if kind == "sparse":      # a handful of nodes per tile: groups span many rows
        return wl.uniform_nodes(5 * (Ms // 16) ** 2 + 3, 2, 3)
    if kind == "crowded":     # one tile of three work items and a remainder
        return 0.2 / 16 * wl.uniform_nodes(2 * 256 + 37, 2, 4) + 0.11
    x = wl.uniform_nodes(997, 2, 5)   # grid lines: columns, rows, both, and the wrap
    x[::3, 0] = np.round(x[::3, 0] * Ms) / Ms
    x[::5, 1] = np.round(x[::5, 1] * Ms) / Ms
    x[0] = [-0.5, -0.5]
    return x


@pytest.mark.parametrize("m", [5, 6, 7, 8])
@pytest.mark.parametrize("kind,M,nrhs", [("one", 32, 1), ("sparse", 64, 2), ("crowded", 32, 5),
                                         ("lines", 32, 1), ("lines", 16, 4)])
def test_window_sums(m, kind, M, nrhs):
    from paper_2302_00414_amd.nfft import Plan
    x = _nodes(kind, 2 * M)
    print(f"[case] {kind} N={x.shape[0]} M={M} m={m} rhs={nrhs}", flush=True)
    p = Plan(x, M, 2.0, m, precision="f32", max_rhs=nrhs)
    h = wl.complex_normal((nrhs, M * M), 7).astype(np.complex64)
    got = p.forward(torch.from_numpy(h).cuda()).cpu().numpy()
    for r in range(nrhs):
        want = onfft.forward(x, h[r].astype(np.complex128), M, 2.0, m)
        assert metrics.rel_err(got[r], want) <= TOL, (kind, m, r)


def _nodes3(kind, Ms):
    if kind == "one":
        return np.array([[0.123, -0.4567, 0.31]])
    if kind == "sparse":      # a few nodes per tile: groups span every plane
        return wl.uniform_nodes(3 * (Ms // 8) ** 3 + 3, 3, 3)
    if kind == "crowded":     # one tile of three work items and a remainder
        return 0.9 * 8 / Ms * wl.uniform_nodes(2 * 256 + 37, 3, 4) + 4.0 / Ms
    x = wl.uniform_nodes(701, 3, 5)   # grid planes of each dimension, and the wrap
    for t in range(3):
        x[t::4, t] = np.round(x[t::4, t] * Ms) / Ms
    x[0] = [-0.5, -0.5, -0.5]
    return x


@pytest.mark.parametrize("m", [4])
@pytest.mark.parametrize("kind,M,nrhs", [("one", 8, 1), ("sparse", 16, 2), ("crowded", 8, 1),
                                         ("lines", 8, 3)])
def test_window_sums_3d(m, kind, M, nrhs):
    from paper_2302_00414_amd.nfft import Plan
    x = _nodes3(kind, 2 * M)
    print(f"[case] 3-D {kind} N={x.shape[0]} M={M} m={m} rhs={nrhs}", flush=True)
    p = Plan(x, M, 2.0, m, precision="f32", max_rhs=nrhs)
    h = wl.complex_normal((nrhs, M ** 3), 7).astype(np.complex64)
    got = p.forward(torch.from_numpy(h).cuda()).cpu().numpy()
    for r in range(nrhs):
        want = onfft.forward(x, h[r].astype(np.complex128), M, 2.0, m)
        assert metrics.rel_err(got[r], want) <= TOL, (kind, m, r)


@pytest.mark.parametrize("m", [5, 6, 7, 8])
@pytest.mark.parametrize("nrhs", [1, 5, 6, 10, 11])
def test_right_hand_sides_of_a_work_group(m, nrhs):
    """256 tiles, one of two work items: with 10 and 11 right-hand sides four
    share a work-group (the last takes two and three), with 5 and 6 two (the last
    one or two)."""
    from paper_2302_00414_amd.nfft import Plan
    M = 128
    x = np.concatenate([wl.uniform_nodes(256 * 24, 2, 8),
                        0.9 * 16 / (2 * M) * wl.uniform_nodes(300, 2, 9) + 8.0 / (2 * M)])
    x[::11, 0] = np.round(x[::11, 0] * 2 * M) / (2 * M)
    x = np.where(x >= 0.5, x - 1.0, x)
    print(f"[case] N={x.shape[0]} M={M} m={m} rhs={nrhs}", flush=True)
    p = Plan(x, M, 2.0, m, precision="f32", max_rhs=nrhs)
    h = wl.complex_normal((nrhs, M * M), 10).astype(np.complex64)
    got = p.forward(torch.from_numpy(h).cuda()).cpu().numpy()
    for r in range(nrhs):
        want = onfft.forward(x, h[r].astype(np.complex128), M, 2.0, m)
        assert metrics.rel_err(got[r], want) <= TOL, (m, r)

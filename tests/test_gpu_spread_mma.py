"""The matrix-core spreading (d = 2, tile edge 16: mode 7 for m <= 7, the default
mode for m = 8, in float32 from 512 tiles on; d = 3, tile edge 8) against the oracle NFFT, at the sizes where
its cuts can go wrong: groups of four and chunks of 64 nodes that are not full, one node,
tiles of several work items, empty tiles and bands, nodes on grid lines (closed
edges; at m = 8 the row edge has its own sums), and right-hand sides that do
not fill the last work-group.

Tolerances (relative l2): float64 differs from the oracle by rounding only,
1e-12; two float32 evaluations in different orders agree to 2e-6, and a float32
transform differs from the oracle by rounding only, 2e-6.
"""
import numpy as np
import pytest
import torch

from oracle import metrics, nfft as onfft
from paper_2302_00414_amd import workloads as wl

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = {"f64": 1e-12, "f32": 2e-6}


def _nodes(kind, Ms):
    if kind == "one":
        return np.array([[0.123, -0.4567]])
    if kind == "sparse":
        return wl.uniform_nodes(5 * (Ms // 16) ** 2 + 3, 2, 3)
    if kind == "crowded":     # most nodes in one tile: several items, full chunks, a remainder
        return np.concatenate([0.9 / Ms * wl.uniform_nodes(1100, 2, 4) * 16 + 8.0 / Ms,
                               wl.uniform_nodes(70, 2, 5)])
    if kind == "row":         # one row of cells: one band, every column
        x = wl.uniform_nodes(519, 2, 6)
        x[:, 0] = (3.0 + 0.9 * (x[:, 0] + 0.5)) / Ms
        return x
    x = wl.uniform_nodes(997, 2, 5)   # grid lines: rows, columns, both, and the wrap
    x[::3, 0] = np.round(x[::3, 0] * Ms) / Ms
    x[::5, 1] = np.round(x[::5, 1] * Ms) / Ms
    x[0] = [-0.5, -0.5]
    return x


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind,M,nrhs", [("one", 16, 1), ("sparse", 64, 2), ("crowded", 16, 5),
                                         ("row", 16, 1), ("lines", 16, 3)])
def test_spreading(prec, m, kind, M, nrhs):
    from paper_2302_00414_amd.nfft import Plan
    x = _nodes(kind, 2 * M)
    N = x.shape[0]
    print(f"[case] {kind} N={N} M={M} m={m} {prec} rhs={nrhs}", flush=True)
    p = Plan(x, M, 2.0, m, precision=prec, max_rhs=nrhs, tuning={"spread_mode": 7} if m <= 7 else None)
    w = (1.0 + 0.5 * wl.complex_normal(N, 8)) / N
    p.set_weights(w)
    f = wl.complex_normal((nrhs, N), 9)
    got = p.adjoint(torch.from_numpy(f).cuda()).cpu().numpy()
    for r in range(nrhs):
        want = onfft.adjoint(x, w * f[r], M, 2.0, m)
        assert metrics.rel_err(got[r], want) <= TOL[prec], (kind, m, r)


@pytest.mark.parametrize("N", [65, 255, 256, 257, 259, 515])
@pytest.mark.parametrize("m", [1, 4, 7])
def test_spreading_of_one_crowded_tile(N, m):
    """One work item of several chunks, float32: the form that stages four
    chunks at a time, at the edges of its 64 and 256 nodes."""
    from paper_2302_00414_amd.nfft import Plan
    M = 16
    x = 0.9 * 16 / 32 * wl.uniform_nodes(N, 2, 4) + 8.0 / 32
    print(f"[case] one tile N={N} M={M} m={m} f32", flush=True)
    p = Plan(x, M, 2.0, m, precision="f32", tuning={"spread_mode": 7, "spread_threads": 64,
                                                    "item_nodes": 512})
    w = (1.0 + 0.5 * wl.complex_normal(N, 8)) / N
    p.set_weights(w)
    f = wl.complex_normal(N, 9)
    got = p.adjoint(torch.from_numpy(f).cuda()).cpu().numpy().reshape(-1)
    assert metrics.rel_err(got, onfft.adjoint(x, w * f, M, 2.0, m)) <= TOL["f32"]


def test_spreading_m8_of_many_tiles():
    """m = 8 in float32 takes the matrix cores from 512 tiles on; nodes on grid
    lines among them."""
    from paper_2302_00414_amd.nfft import Plan
    M, m, N, nrhs = 256, 8, 1024 * 65, 3
    x = wl.uniform_nodes(N, 2, 13)
    x[::7, 0] = np.round(x[::7, 0] * 2 * M) / (2 * M)
    x[::9, 1] = np.round(x[::9, 1] * 2 * M) / (2 * M)
    x = np.where(x >= 0.5, x - 1.0, x)
    print(f"[case] many tiles N={N} M={M} m={m} f32 rhs={nrhs}", flush=True)
    p = Plan(x, M, 2.0, m, precision="f32", max_rhs=nrhs)
    p.set_weights(np.full(N, 1.0 / N))
    f = wl.complex_normal((nrhs, N), 14)
    got = p.adjoint(torch.from_numpy(f).cuda()).cpu().numpy()
    for r in range(nrhs):
        assert metrics.rel_err(got[r], onfft.adjoint(x, f[r] / N, M, 2.0, m)) <= TOL["f32"], r


def _nodes3(kind, Ms):
    if kind == "one":
        return np.array([[0.123, -0.4567, 0.31]])
    if kind == "sparse":      # groups of four span several planes
        return wl.uniform_nodes(3 * (Ms // 8) ** 3 + 3, 3, 3)
    if kind == "crowded":     # one tile of several items, full chunks and a remainder
        return 0.9 * 8 / Ms * wl.uniform_nodes(2 * 256 + 101, 3, 4) + 4.0 / Ms
    x = wl.uniform_nodes(701, 3, 5)   # grid planes of each dimension, and the wrap
    for t in range(3):
        x[t::4, t] = np.round(x[t::4, t] * Ms) / Ms
    x[0] = [-0.5, -0.5, -0.5]
    return x


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [1, 2, 3, 4])
@pytest.mark.parametrize("kind,M,nrhs", [("one", 8, 1), ("sparse", 16, 1), ("crowded", 8, 1),
                                         ("lines", 8, 2)])
def test_spreading_3d(prec, m, kind, M, nrhs):
    from paper_2302_00414_amd.nfft import Plan
    x = _nodes3(kind, 2 * M)
    N = x.shape[0]
    print(f"[case] 3-D {kind} N={N} M={M} m={m} {prec} rhs={nrhs}", flush=True)
    w = (1.0 + 0.5 * wl.complex_normal(N, 8)) / N
    f = wl.complex_normal((nrhs, N), 9)
    for tuning in ({"spread_mode": 7}, None):
        p = Plan(x, M, 2.0, m, precision=prec, max_rhs=nrhs, tuning=tuning)
        p.set_weights(w)
        got = p.adjoint(torch.from_numpy(f).cuda()).cpu().numpy()
        for r in range(nrhs):
            want = onfft.adjoint(x, w * f[r], M, 2.0, m)
            assert metrics.rel_err(got[r], want) <= TOL[prec], (kind, m, r, tuning)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nrhs", [2, 7])
def test_right_hand_sides_share_the_factors(prec, nrhs):
    """Enough work-groups for several right-hand sides each: the same bits as
    one at a time (every cell's sum has one order)."""
    from paper_2302_00414_amd.nfft import Plan
    M, m, N = 256, 6, 140003
    x = wl.uniform_nodes(N, 2, 11)
    p = Plan(x, M, 2.0, m, precision=prec, max_rhs=nrhs, tuning={"spread_mode": 7})
    p.set_weights(np.full(N, 1.0 / N))
    f = torch.from_numpy(wl.complex_normal((nrhs, N), 12)).to(p.cdtype).cuda()
    both = p.adjoint(f)
    one = torch.stack([p.adjoint(f[r]) for r in range(nrhs)])
    rel = ((both - one).norm() / one.norm()).item()
    assert rel <= {"f64": 1e-14, "f32": 1e-6}[prec], rel

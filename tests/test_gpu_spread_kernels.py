"""Every spreading kernel that a plan can be asked for, by name: the LDS kernels
with the mode set to 1 (a default plan leaves the kernel to the library), the
matrix-core kernels of mode 7 with each thread count and with two right-hand
sides a work-group, and the tile kernel at m = 8, which only the default mode
takes, on sets that reach it. Nodes on grid lines (closed edges), a crowded tile
of several work items with a remainder, and empty tiles are in every set.

Tolerances (relative l2), as in the tests of the same kernels elsewhere: against
the oracle float64 1e-12 and float32 2e-6; two kernels against one another
float64 1e-13 and float32 2e-6; the float64 LDS kernels among themselves, which
differ in the order of their atomics only, 1e-14.
"""
import numpy as np
import pytest
import torch

from oracle import metrics, nfft as onfft
from paper_2302_00414_amd import workloads as wl

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = {"f64": 1e-12, "f32": 2e-6}
TOL_ORDER = {"f64": 1e-13, "f32": 2e-6}


def _nodes(d, N, Ms, seed, crowd=700):
    """N uniform nodes (every seventh on a grid line of dimension 0, every ninth of
    the last one) in three quarters of dimension 0, and `crowd` in one tile."""
    T = 16 if d == 2 else 8
    x = wl.uniform_nodes(N, d, seed)
    x[:, 0] = 0.75 * x[:, 0]
    x[::7, 0] = np.round(x[::7, 0] * Ms) / Ms
    x[::9, -1] = np.round(x[::9, -1] * Ms) / Ms
    x = np.concatenate([x, 0.9 * T / Ms * wl.uniform_nodes(crowd, d, seed + 1) + 0.5 * T / Ms])
    return np.where(x >= 0.5, x - 1.0, x)


def _run(x, M, m, prec, F, w, tuning):
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] N={x.shape[0]} d={x.shape[1]} M={M} m={m} {prec} rhs={F.shape[0]} {tuning}", flush=True)
    p = Plan(x, M, 2.0, m, precision=prec, max_rhs=F.shape[0], tuning=tuning)
    p.set_weights(w)
    Ft = torch.from_numpy(F)
    got = [p.adjoint(Ft).cpu().numpy() for _ in range(2)]
    p.close()
    return got


def _data(x, nrhs, seed):
    N = x.shape[0]
    return (1.0 + 0.3 * wl.complex_normal(N, seed)) / N, wl.complex_normal((nrhs, N), seed + 1)


def _check(got, x, w, F, M, m, tol):
    for r in range(F.shape[0]):
        assert metrics.rel_err(got[r], onfft.adjoint(x, w * F[r], M, 2.0, m)) <= tol, r


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("nt", [64, 256, 512])
@pytest.mark.parametrize("items", [64, 600])
def test_mode7_float32_of_one_right_hand_side(m, nt, items):
    """64 threads: the tile kernel; 256 and 512: four and eight waves with a
    padded tile each."""
    M = 32
    x = _nodes(2, 1500, 2 * M, 700 + m)
    w, F = _data(x, 1, 710)
    got, again = _run(x, M, m, "f32", F, w, {"spread_mode": 7, "spread_threads": nt, "item_nodes": items})
    lds, _ = _run(x, M, m, "f32", F, w, {"spread_mode": 1, "item_nodes": items})
    assert np.array_equal(got, again)
    assert not np.array_equal(got, lds)   # another kernel did run
    _check(got, x, w, F, M, m, TOL["f32"])
    assert metrics.rel_err(got[0], lds[0]) <= TOL_ORDER["f32"]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [1, 2, 3, 4])
def test_lds_kernel_3d(m, prec):
    M = 16
    x = _nodes(3, 1500, 2 * M, 720 + m)
    w, F = _data(x, 2, 730)
    lds, _ = _run(x, M, m, prec, F, w, {"spread_mode": 1})
    mma, _ = _run(x, M, m, prec, F, w, {"spread_mode": 7})
    _check(lds, x, w, F, M, m, TOL[prec])
    for r in range(2):
        assert metrics.rel_err(mma[r], lds[r]) <= TOL_ORDER[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 7, 8])
def test_lds_kernel_and_its_window_sources(m, prec):
    """Mode 1 evaluates the window before the nodes are spread, 3 reads it from a
    table, 4 evaluates it late: the same values, added in the same order."""
    M = 32
    x = _nodes(2, 1500, 2 * M, 740 + m)
    w, F = _data(x, 2, 750)
    one, _ = _run(x, M, m, prec, F, w, {"spread_mode": 1})
    _check(one, x, w, F, M, m, TOL[prec])
    for mode in (3, 4):
        other, _ = _run(x, M, m, prec, F, w, {"spread_mode": mode})
        for r in range(2):
            assert metrics.rel_err(other[r], one[r]) <= {"f64": 1e-14, "f32": 1e-7}[prec], mode


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [1, 3, 4, 6, 7])
@pytest.mark.parametrize("nrhs", [5, 6])
def test_two_right_hand_sides_a_work_group(m, nrhs, prec):
    """More than 512 pairs of a work item and two right-hand sides, the last pair
    full and half full."""
    M = 128
    x = _nodes(2, 192 * 20, 2 * M, 760 + m)
    w, F = _data(x, nrhs, 770)
    got, again = _run(x, M, m, prec, F, w, {"spread_mode": 7, "spread_threads": 64})
    assert np.array_equal(got, again)
    _check(got, x, w, F, M, m, TOL[prec])


@pytest.mark.parametrize("prec,M,N,nrhs", [
    ("f64", 16, 1060, 1),                # four tiles, one item each once joined
    ("f64", 16, 1060, 3),
    ("f64", 256, 768 * 130, 1), ("f64", 128, 192 * 150, 3),
    ("f32", 128, 192 * 80, 4), ("f32", 256, 768 * 70, 1)])
def test_tile_kernel_at_m8(prec, M, N, nrhs):
    m = 8
    x = _nodes(2, N, 2 * M, 780, crowd=0 if M == 16 else 700)
    if M == 16:
        x[:, 0] = x[:, 0] / 0.75          # all four tiles
        x = np.where(x >= 0.5, x - 1.0, x)
    w, F = _data(x, nrhs, 790)
    got, again = _run(x, M, m, prec, F, w, None)
    assert np.array_equal(got, again)     # the float64 LDS kernel's atomics do not repeat
    if prec == "f32":
        assert not np.array_equal(got, _run(x, M, m, prec, F, w, {"spread_mode": 1})[0])
    _check(got, x, w, F, M, m, TOL[prec])

"""Float32 error of the matrix-core spreading against the LDS kernel's.

Both evaluate the same window polynomials and differ in the order of their sums
only, so on the same inputs the errors of their transforms against float64 agree
but for the rounding of the factors. Emulated in float32 with fused operations,
the factors' rms errors lie within 5 % of a Horner chain's when the constant
term enters last and 12 to 25 % above it when it enters inside the even chain; of
the transform's error (in squares) the factors make about a third, the FFT and
the sums the rest: 2 % separates the two.
"""
import numpy as np
import pytest
import torch

from paper_2302_00414_amd import workloads as wl

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,M,N,m", [(3, 32, 65536, 2), (3, 16, 12800, 3), (3, 32, 65536, 3),
                                     (3, 16, 1280, 4), (2, 64, 3000, 4), (2, 128, 40321, 6)])
def test_float32_error_is_the_lds_kernels(d, M, N, m):
    from paper_2302_00414_amd.nfft import Plan
    print(f"[case] d={d} M={M} N={N} m={m} f32", flush=True)
    x = wl.uniform_nodes(N, d, 1)
    w = np.full(N, 1.0 / N)
    exact = Plan(x, M, 2.0, m, precision="f64")
    plans = [Plan(x, M, 2.0, m, precision="f32", tuning={"spread_mode": mode, "spread_threads": 64})
             for mode in (1, 7)]
    err = np.zeros(2)
    for p in (exact, *plans):
        p.set_weights(w)
    for seed in range(8):
        v = torch.from_numpy(wl.complex_normal(N, 20 + seed)).to(torch.complex64).cuda()
        want = exact.adjoint(v.to(torch.complex128))
        for k, p in enumerate(plans):
            got = p.adjoint(v).to(torch.complex128)
            err[k] += (((got - want).norm() / want.norm()) ** 2).item()
    lds, mma = np.sqrt(err / 8)
    print(f"[error] LDS {lds:.3e} matrix cores {mma:.3e}", flush=True)
    assert mma <= 1.02 * lds, (mma, lds)
    for p in (exact, *plans):
        p.close()

"""Rate coefficients at temperatures far below the energies' spacing (GPU): (interval / beta)^4
passes the range of doubles and the Boltzmann factor is zero beyond the threshold.  There the
integral is its leading terms at the threshold, in closed form: with s(th + x) = s0 + s1 x,
  int s(U) U e^{-(U - th)/beta} dU = beta (s0 th) + beta^2 (s0 + s1 th) + 2 beta^3 s1 + ...,
further terms being smaller by beta / spacing < 1e-50.  Rounding of some ten operations: 1e-14
relative; 1e-12 allowed."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = np.array([0.002, 0.004, 0.007])
# level energies: pairs (1, 0) and (2, 0) start on the ramp, (0, 0) at threshold 0, (3, 0) has
# its threshold between the first two energies, (4, 0) beyond the last
E = np.array([0.0, 0.0011, 0.003, 0.006, 0.02])
MU = 2000.0


def natural_cubic(y):
    h0, h1 = np.diff(U)
    m = ((y[2] - y[1]) / h1 - (y[1] - y[0]) / h0) / ((h0 + h1) / 3.0)
    return lambda x: (y[0] + ((y[1] - y[0]) / h0 - h0 * m / 6.0) * x + m / (6.0 * h0) * x ** 3,
                      (y[1] - y[0]) / h0 - h0 * m / 6.0 + m / (2.0 * h0) * x ** 2)


@pytest.mark.parametrize("beta", [1e-60, 1e-85, 1e-95])
def test_cold_limit(gpu_lib, beta):
    print("[gpu] rates beta=%g" % beta, flush=True)
    ctx = gpu_lib.Context()
    rng = np.random.default_rng(2)
    sym = rng.random((3, 5, 5)) + 1.0
    sym = sym + np.swapaxes(sym, 1, 2)
    k = ctx.rate_coefficients(U, sym, E, np.ones(5), MU, np.array([beta, 1e-3]))
    ctx.close()
    assert np.all(np.isfinite(k))
    for i in range(1, 5):
        th, y = 0.5 * E[i], sym[:, i, 0]
        if th < U[0]:
            s0, s1 = 0.0, y[0] / (U[0] - th)
        elif th < U[-1]:
            s0, s1 = natural_cubic(y)(th - U[0])
        else:
            s0, s1 = y[-1], 0.0
        # (beta^-3/2) beta = beta^-1/2 first, so that no factor leaves the range
        ref = np.sqrt(8.0 / (np.pi * MU)) * beta ** -0.5 * (
            s0 * th + beta * (s0 + s1 * th) + 2.0 * beta * beta * s1)
        assert abs(k[0, i, 0] / ref - 1.0) < 1e-12, i
    ref = np.sqrt(8.0 / (np.pi * MU)) * 2.0 * beta ** 1.5 * sym[0, 0, 0] / U[0]
    assert abs(k[0, 0, 0] / ref - 1.0) < 1e-12
    assert np.all(k[0, 0, 1:] == 0.0)          # uphill: exp(-dE / beta)

"""Cross sections and rates at the edges of their kernels' tilings (GPU).

* cross sections: trajectory counts around the 1024-entry list chunk, levels around
  the 64-lane tile, rows that fit LDS and rows that do not, an empty level, against
  the oracle.  Sums of positive terms: 1e-13 relative.
* rates: 2, 3, 17 and 64 energies, 1, 4 and 5 temperatures, level counts that leave a
  partial workgroup, beta from far below to far above the energy spacing (both forms
  of the moments), against the oracle's adaptive quadrature: 1e-10 relative.
"""
import sys

import numpy as np
import pytest

import oracle
from oracle import postproc as PP

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.synchronize()
    c.close()


@pytest.mark.parametrize("B,N,nl", [(1, 1, 1), (255, 65, 64), (1024, 97, 65), (1025, 130, 3),
                                    (2500, 33, 200), (70, 4096, 129), (9, 4097, 40)])
def test_cross_sections_edges(ctx, B, N, nl):
    import torch
    print("[gpu] xsec B=%d N=%d levels=%d" % (B, N, nl), flush=True)
    rng = np.random.default_rng(B + N)
    P = rng.random((B, N))
    b = rng.uniform(0.0, 20.0, B)
    lev = rng.integers(0, nl, N).astype(np.int32)
    init = rng.integers(0, max(1, nl - 1), B).astype(np.int32)      # the last level stays empty
    sig = ctx.cross_sections(torch.as_tensor(P, device=ctx.device), b, init, lev, nl, 20.0)
    ref = oracle.cross_sections(init, b, P, lev, nl, 20.0)
    sys.stdout.flush()
    assert np.allclose(sig.cpu().numpy(), ref, rtol=1e-13, atol=0.0)


@pytest.mark.parametrize("nE,nT,L", [(2, 1, 1), (3, 4, 7), (17, 5, 13), (64, 1, 12)])
def test_rates_edges(ctx, nE, nT, L):
    print("[gpu] rates nE=%d nT=%d L=%d" % (nE, nT, L), flush=True)
    rng = np.random.default_rng(nE)
    U = np.sort(rng.uniform(1e-4, 0.05, nE))
    E = rng.uniform(0.0, 0.03, L)
    g = rng.integers(1, 9, L).astype(float)
    sym = rng.random((nE, L, L)) * 20.0 + 1.0
    gap = np.diff(U).mean()
    beta = gap * np.array([3e-2, 30.0, 0.3, 3.0, 0.1])[:nT]
    pairs = [tuple(x) for x in rng.integers(0, L, (min(L * L, 12), 2))]
    k = ctx.rate_coefficients(U, sym, E, g, 2000.0, beta)
    k_o = PP.rate_coefficients(U, sym, E, g, 2000.0, beta, pairs=pairs)
    k_s = np.stack([k[:, i, f] for i, f in pairs], axis=1)
    big = np.abs(k_o) > 1e-290
    assert np.max(np.abs(k_s[big] - k_o[big]) / np.abs(k_o[big])) < 1e-10

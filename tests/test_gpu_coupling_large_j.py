"""The coupling fill with its m-coefficients at the edge of 64 KiB of LDS and at their largest
(GPU): total j = 40 with lam up to 39, and the largest angular momenta the builder takes, j1 =
j2 = 40, lam = 40.  Against the screened builder's values, which read the same factors by another
kernel without LDS: sums of up to 9 products in another order, 9 eps = 2e-15 of the sum of
magnitudes; 1e-13 of the largest element allowed."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jr,lmax", [(20, 39), (20, 40), (40, 40), (6, 40)])
def test_dense_equals_screened(gpu_lib, jr, lmax):
    import torch
    print("[gpu] coupling j1 = j2 = %d, lam <= %d" % (jr, lmax), flush=True)
    rng = np.random.default_rng(jr)
    rj = np.array([jr - 1, jr], np.int32)
    b = np.zeros((2, 2 * jr + 1))
    for r in range(2):
        b[r, :2 * rj[r] + 1] = rng.standard_normal(2 * rj[r] + 1)
        b[r] /= np.linalg.norm(b[r])
    ch = [(r, j2, j, m) for m in (-1, 0, 2) for r in range(2) for j2 in (jr - 1, jr)
          for j in range(rj[r] + j2 - 2, rj[r] + j2 + 1)]
    col = lambda i: np.array([c[i] for c in ch], np.int32)
    basis = types.SimpleNamespace(rot1=col(0), j2=col(1), j=col(2), m=col(3), rot1_j=rj, b=b)
    terms = [(0, 0, 0, 0), (2, 0, 0, 2), (2, 2, 2, 2), (3, 1, 2, 4), (4, 0, 4, 6), (8, 2, 6, 10),
             (20, 0, 20, 38), (20, 2, 20, lmax), (20, 1, 19, 39)]
    t = np.array(terms, np.int32)
    ex = types.SimpleNamespace(lam1=t[:, 0], mu1=t[:, 1], lam2=t[:, 2], lam=t[:, 3],
                               v=rng.uniform(0.5, 1.5, (len(t), 19)))
    ctx = gpu_lib.Context()
    M = ctx.build_couplings(basis, ex)["M"]
    sp = ctx.build_couplings_sparse(basis, ex, np.ascontiguousarray(ex.v[:, :2]), 0.0)
    S = torch.zeros_like(M)
    S[:, sp["rows"].long(), sp["cols"].long()] = sp["values"]
    ctx.close()
    big = float(M.abs().max())
    assert np.isfinite(big) and big > 0 and sp["n_kept"] > 0
    assert float((M - S).abs().max()) < 1e-13 * big

"""The coupling fill at the edges of its tiles (GPU): one term to one more than the staged
terms, one knot to more than two knot ranges, groups of one channel to more than a wave's,
both channel orders, tables and angular factors alone and together.  Against the oracle's Eq. 17 sums, to 1e-13 of the largest element as for the
builder's other tests (sums of up to 97 products: 97 eps = 2e-14).
"""
import numpy as np
import pytest

import oracle
from synth import coupling as C

pytestmark = pytest.mark.gpu

TERMS = [(l1, mu1, l2, l) for l1 in range(5) for mu1 in range(l1 + 1) for l2 in range(3)
         for l in range(abs(l1 - l2), l1 + l2 + 1)]


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.synchronize()
    c.close()


@pytest.mark.parametrize("T,K,j1,order", [
    (1, 1, 0, "m"), (2, 15, 1, "level"), (15, 16, 1, "m"), (16, 17, 1, "level"),
    (17, 63, 1, "m"), (95, 64, 1, "m"), (96, 65, 1, "level"), (97, 129, 1, "m"),
    (81, 33, 2, "m"), (9, 7, 3, "m")])
def test_fill_edges(ctx, T, K, j1, order):
    import torch
    rng = np.random.default_rng(T * 131 + K)
    basis = C.top_rotor_basis(j1, (0, 1, 2), order=order)
    terms = [TERMS[i] for i in np.sort(rng.permutation(len(TERMS))[:T])]
    ex = C.synthetic_expansion(terms, np.linspace(4.0, 20.0, K), seed=5)
    print("[gpu] fill T=%d K=%d N=%d %s" % (T, K, basis.N, order), flush=True)
    M_o, G_o = oracle.coupling_tables(basis, ex)
    both = ctx.build_couplings(basis, ex, tables=True, angular=True)
    M1 = ctx.build_couplings(basis, ex)["M"]
    G1 = ctx.build_couplings(basis, ex, tables=False, angular=True)["G"]
    assert torch.equal(M1, both["M"]) and torch.equal(G1, both["G"])
    assert np.max(np.abs(M1.cpu().numpy() - M_o)) < 1e-13 * max(np.abs(M_o).max(), 1e-300)
    assert np.max(np.abs(G1.cpu().numpy() - G_o)) < 1e-13 * max(np.abs(G_o).max(), 1e-300)

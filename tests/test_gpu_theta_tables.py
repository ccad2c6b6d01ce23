"""Tables from potential coefficients and the gradient's sum over the batch (GPU).

The tables that set_theta builds against tables summed on the host, through a propagation
(1e-12 of a probability: 16 digits over some hundred stages): knot counts around the
builder's chunk of 16, elements around its 256, one angular term to 48, up to 256
coefficients, dense and sparse tables, and more bytes than stay with the context.  The
gradient of a batch against the sum of its parts (B eps of the largest entry: 1e-12).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.synchronize()
    c.close()


def model(N, K, nG, P, fill, seed=3):
    rng = np.random.default_rng(seed + 1000 * N + K)
    G = rng.normal(size=(nG, N, N)) * (rng.random((nG, N, N)) < fill)
    G = np.triu(G) + np.triu(G, 1).transpose(0, 2, 1)
    R = np.linspace(3.0, 30.0, K)
    gidx = np.concatenate([np.arange(nG), rng.integers(0, nG, P - nG)]).astype(np.int32)
    rad = np.exp(-(R[None] - rng.uniform(3.0, 9.0, P)[:, None]) ** 2 / 8.0)
    theta = 1e-3 * rng.normal(size=P)
    M = np.einsum("tk,tnm->knm", np.stack([(theta * (gidx == t)) @ rad for t in range(nG)]), G)
    return dict(R=R, E=np.sort(rng.uniform(0.0, 5e-3, N)), G=G, gidx=gidx, rad=rad, theta=theta, M=M)


def batch(B, N, steps=12):
    rng = np.random.default_rng(B)
    R0 = rng.uniform(6.0, 25.0, B)
    return dict(init_channel=rng.integers(0, N, B).astype(np.int32), E_coll=rng.uniform(1e-3, 8e-3, B),
                b=rng.uniform(0.0, 0.8, B) * R0, R0=R0, dt=np.full(B, 20.0), n_steps=np.full(B, steps))


@pytest.mark.parametrize("N,K,nG,P,layout", [
    (1, 4, 1, 1, "dense"), (15, 15, 1, 3, "dense"), (16, 16, 2, 2, "dense"), (17, 17, 12, 96, "sparse"),
    (33, 33, 48, 256, "sparse"), (81, 47, 12, 96, "dense"), (640, 210, 2, 4, "dense")])
def test_tables_and_gradient_sum(ctx, N, K, nG, P, layout):
    print("[gpu] theta tables N=%d K=%d nG=%d P=%d %s" % (N, K, nG, P, layout), flush=True)
    s = model(N, K, nG, P, 1.0 if layout == "dense" else 0.3)
    kw = dict(R_grid=s["R"], E=s["E"], mu=3000.0, storage="R64", layout=layout)
    ref = ctx.load_system(M=s["M"], **kw)
    sid = ctx.load_system(M=s["M"], **kw)
    ctx.set_params(sid, s["rad"], s["gidx"], s["G"])
    ctx.set_theta(sid, 2.0 * s["theta"])
    ctx.set_theta(sid, s["theta"])
    B = 12
    b = batch(B, N)
    P0 = ctx.run_host([ref] * B, [N] * B, schedule="gemv", **b)["P"]
    P1 = ctx.run_host([sid] * B, [N] * B, schedule="gemv", **b)["P"]
    assert np.max(np.abs(P0 - P1)) < 1e-12
    if N <= 81:
        for B in (1, 255, 300):
            b = batch(B, N, 3)
            w = np.random.default_rng(1).normal(size=(B, N))
            g, _ = ctx.adjoint(sid, N, w, n_param=P, **b)
            h = B // 2
            parts = np.zeros(P)
            for q in (slice(0, h), slice(h, B)):
                if q.stop > q.start:
                    parts += ctx.adjoint(sid, N, w[q], n_param=P, **{k: v[q] for k, v in b.items()})[0]
            assert np.max(np.abs(g - parts)) <= 1e-12 * np.max(np.abs(g))
    ctx.free_system(ref)
    ctx.free_system(sid)

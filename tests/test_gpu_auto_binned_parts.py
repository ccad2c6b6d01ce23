"""Fixed-step batches that the default schedule sends to the knot-binned products, in parts
(GPU): a ragged run in two calls with complex tables, and with amplitudes too long for the
combine's LDS (Npad > 2048); a batch of several passes, also when there is no room for the
first size of a pass.  Each is the run in one piece bit for bit: the route depends on the
system and the batch and not on step counts, and a trajectory's products not on its
neighbours."""
import os
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def system(N, K, cplx):
    rng = np.random.default_rng(N)
    R = np.linspace(4.0, 20.0, K)
    H = rng.standard_normal((2, N, N)) + (1j * rng.standard_normal((2, N, N)) if cplx else 0)
    H = 0.5 * (H + np.conj(np.swapaxes(H, 1, 2)))
    f = np.stack([1e-5 * np.exp(-0.2 * R), 1e-5 * np.cos(R)])
    return types.SimpleNamespace(N=N, R=R, E=np.sort(rng.uniform(0.0, 9e-3, N)), mu=12000.0,
                                 M=np.einsum("qk,qnm->knm", f, H))


def load(ctx, s, storage):
    return ctx.load_system(R_grid=s.R, E=s.E, M=s.M, mu=s.mu, storage=storage)


def batch(s, steps):
    B = len(steps)
    rng = np.random.default_rng(3)
    c0 = np.zeros((B, 6))
    k = np.sqrt(2 * s.mu * rng.uniform(1e-3, 6e-3, B))
    c0[:, 0], c0[:, 1], c0[:, 3] = rng.uniform(5.0, 19.0, B), 0.5 * np.pi, -k
    c0[:, 5] = rng.uniform(0.0, 2.0, B) * k
    return dict(init_channel=rng.integers(0, s.N, B).astype(np.int32), classical0=c0,
                dt=np.full(B, 8.0), n_steps=np.asarray(steps))


def launches_of(ctx, f):
    ctx.set_profiling(True)
    ctx.profile_read()
    out = f()
    n = ctx.profile_read()[1]
    ctx.set_profiling(False)
    return out, n


@pytest.mark.parametrize("N,K,cplx", [(365, 12, True), (2050, 4, False), (2050, 4, True)])
def test_two_calls_equal_one(gpu_lib, N, K, cplx):
    print("[gpu] auto binned in two calls N=%d complex=%d" % (N, cplx), flush=True)
    s = system(N, K, cplx)
    ctx = gpu_lib.Context()
    sid = load(ctx, s, "C128" if cplx else "R64")
    steps, first = np.array([9, 4, 0, 9]), np.array([5, 4, 0, 1])
    kw = batch(s, steps)
    ids, Ns = [sid] * 4, [N] * 4
    one, n = launches_of(ctx, lambda: ctx.run_host(ids, Ns, **kw))
    assert n == 4 * 9 + 1
    ctx.run_host(ids, Ns, **dict(kw, n_steps=first))
    two = ctx.run_host(ids, Ns, n_steps=steps - first, resume=True)
    for f in ("P", "a_final", "classical", "t_final", "steps", "status"):
        assert np.array_equal(one[f], two[f]), f
    ctx.close()


def test_passes_equal_one_pass(gpu_lib):
    print("[gpu] auto binned passes", flush=True)
    s = system(170, 64, True)
    B = 1000
    kw = batch(s, np.random.default_rng(1).integers(0, 4, B))
    out = {}
    for passes in (1, 2):
        ctx = gpu_lib.Context()
        sid = load(ctx, s, "C128")
        ids, Ns = [sid] * B, [s.N] * B
        ctx.run_host(ids, Ns, schedule="gemv", **kw)      # every other buffer is there
        if passes == 2:      # the workspace is refused once: half the trajectories at a time
            os.environ["MQCT_FAULT"] = "alloc@01"
        try:
            out[passes], n = launches_of(ctx, lambda: ctx.run_host(ids, Ns, **kw))
        finally:
            os.environ.pop("MQCT_FAULT", None)
        assert n == passes * (4 * 3 + 1)
        ctx.close()
    for f in ("P", "a_final", "classical", "t_final", "steps", "status", "energy_err"):
        assert np.array_equal(out[1][f], out[2][f]), f

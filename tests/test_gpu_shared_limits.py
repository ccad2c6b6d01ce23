"""Where the default schedule leaves the shared-stream form, and what that form does with a
trajectory that blows up (GPU).  Which kernel ran is read from the bits: the per-trajectory
schedule's own kernel gives its results exactly, the shared-stream form other roundings."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def banded(N, cplx, band=8, K=20):
    rng = np.random.default_rng(N)
    R = np.linspace(4.0, 20.0, K)
    H = rng.standard_normal((N, N)) + (1j * rng.standard_normal((N, N)) if cplx else 0)
    i = np.arange(N)
    H = np.where(np.abs(i[:, None] - i[None]) <= band, 0.5 * (H + np.conj(H.T)), 0)
    return types.SimpleNamespace(N=N, R=R, E=np.sort(rng.uniform(0.0, 9e-3, N)), mu=12000.0,
                                 M=(1e-5 * np.exp(-0.2 * R))[:, None, None] * H)


def batch(s, B, steps):
    rng = np.random.default_rng(3)
    c0 = np.zeros((B, 6))
    k = np.sqrt(2 * s.mu * rng.uniform(1e-3, 6e-3, B))
    c0[:, 0], c0[:, 1], c0[:, 3] = rng.uniform(6.0, 18.0, B), 0.5 * np.pi, -k
    c0[:, 5] = rng.uniform(0.0, 2.0, B) * k
    return dict(init_channel=rng.integers(0, s.N, B).astype(np.int32), classical0=c0,
                dt=np.full(B, 8.0), n_steps=np.full(B, steps))


# N, complex, storage, most trajectories per compute unit in the shared-stream form
CASES = [(120, True, "C128", 2), (160, True, "C128", 2), (176, True, "C128", 1),
         (256, False, "R64", 2), (336, False, "R64", 2), (352, False, "R64", 1),
         (512, False, "R64", 1), (400, False, "R32", 2), (520, False, "R64", 0)]


@pytest.mark.parametrize("N,cplx,storage,per_unit", CASES)
def test_most_trajectories(gpu_lib, N, cplx, storage, per_unit):
    import torch
    print("[gpu] shared limits N=%d %s" % (N, storage), flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    s = banded(N, cplx)
    ctx = gpu_lib.Context()
    sid = ctx.load_system(R_grid=s.R, E=s.E, M=s.M, mu=s.mu, storage=storage, layout="sparse")
    tol = 1e-12 if storage in ("R64", "C128") else 1e-6
    for B, shared in ((max(per_unit, 1) * cus, per_unit > 0), (per_unit * cus + 1, False)):
        kw = batch(s, B, 6)
        a = ctx.run_host([sid] * B, [N] * B, **kw)["a_final"]
        g = ctx.run_host([sid] * B, [N] * B, schedule="gemv", **kw)["a_final"]
        assert np.array_equal(a, g) != shared, B
        assert np.max(np.abs(a - g)) < tol
    ctx.close()


# dense tables: N, complex, storage, trajectories per compute unit above one (fraction),
# shared-stream form?
BYTES = [(121, False, "R64", 0.01, True), (121, False, "R64", 0.5, False),
         (176, False, "R64", 0.0, True), (160, True, "C64", 0.01, True),
         (160, True, "C64", 0.1, False), (112, True, "C128", 0.4, True)]


@pytest.mark.parametrize("N,cplx,storage,more,shared", BYTES)
def test_most_bytes(gpu_lib, N, cplx, storage, more, shared):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the sizes are those of 256 compute units")
    B = cus + int(more * cus)
    print("[gpu] shared bytes N=%d %s B=%d" % (N, storage, B), flush=True)
    s = banded(N, cplx, band=N)
    ctx = gpu_lib.Context()
    sid = ctx.load_system(R_grid=s.R, E=s.E, M=s.M, mu=s.mu, storage=storage)
    kw = batch(s, B, 4)
    a = ctx.run_host([sid] * B, [N] * B, **kw)["a_final"]
    g = ctx.run_host([sid] * B, [N] * B, schedule="gemv", **kw)["a_final"]
    ctx.close()
    assert np.array_equal(a, g) != shared
    assert np.max(np.abs(a - g)) < (1e-12 if storage in ("R64", "C128") else 1e-6)


@pytest.mark.parametrize("schedule", ["auto", "queue"])
@pytest.mark.parametrize("N,cplx,storage", [(9, False, "R64"), (49, True, "C64"), (140, True, "C128")])
def test_blow_up(gpu_lib, N, cplx, storage, schedule):
    """A step of 1e300 atomic units leaves one trajectory non-finite at once: it stops there and
    is flagged as on the per-trajectory schedule, and its neighbours run on."""
    print("[gpu] shared blow-up N=%d %s %s" % (N, storage, schedule), flush=True)
    s = banded(N, cplx, band=N)
    ctx = gpu_lib.Context()
    ctx.set_option("autotune", 0)
    ctx.set_option("tail", 2)
    sid = ctx.load_system(R_grid=s.R, E=s.E, M=s.M, mu=s.mu, storage=storage)
    kw = batch(s, 5, 7)
    kw["dt"][2] = 1e300
    kw["n_steps"][4] = 0
    g = ctx.run_host([sid] * 5, [N] * 5, schedule=schedule, **kw)
    ref = ctx.run_host([sid] * 5, [N] * 5, schedule="gemv", **kw)
    ctx.close()
    assert ref["status"][2] & 16 and ref["steps"][2] < 7
    assert np.array_equal(g["status"], ref["status"]) and np.array_equal(g["steps"], ref["steps"])
    assert np.array_equal(g["t_final"], ref["t_final"])
    ok = [0, 1, 3, 4]
    tol = 1e-12 if storage in ("R64", "C128") else 1e-6
    for f, n in (("P", N), ("a_final", N), ("classical", 6)):
        d = np.abs(g[f] - ref[f]).reshape(5, n)[ok] / (1 + np.abs(ref[f]).reshape(5, n)[ok])
        assert np.max(d) < tol, f
    assert not np.all(np.isfinite(g["P"].reshape(5, N)[2]))

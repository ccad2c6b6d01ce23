"""Fixed-step batches that the default schedule sends to the knot-binned products (GPU).

The library's choice against the per-trajectory kernels: real and complex FP64 tables on
both sides of the choice's lines, ragged step counts with zero, start amplitudes, AT
dynamics, paths off the grid at both ends, a trajectory that blows up, a resumed run, a
batch of several passes, and a device without room for the workspace.  Which schedule ran
is read from the number of timed launches: one per-trajectory launch, or a product per
stage.  The two differ in the order of FP64 sums of up to 2 N terms: 2 N eps = 2.3e-13 a
stage at N = 1030, over at most 45 stages 1e-11; 1e-10 allowed.
"""
import os

import numpy as np
import pytest

from synth import systems as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.synchronize()
    c.close()


def system(N, K, cplx):
    s = S.large_random_system(N=N, K=K, cfg_index=37, workers=0)
    if not cplx:
        s.M = np.ascontiguousarray(s.M.real)
    return s


def batch(s, B, steps, kind=""):
    rng = np.random.default_rng(11)
    R0 = rng.uniform(s.R_grid[1] + 0.5, s.R_grid[-1] - 0.5, B)
    c0 = np.zeros((B, 6))
    k = np.sqrt(2 * s.mu * rng.uniform(1e-3, 6e-3, B))
    c0[:, 0], c0[:, 1], c0[:, 3] = R0, 0.5 * np.pi, -k
    c0[:, 5] = rng.uniform(0.0, 2.0, B) * k
    n = np.full(B, steps)
    kw = dict(init_channel=rng.integers(0, s.N, B).astype(np.int32), classical0=c0,
              dt=np.full(B, 8.0), n_steps=n)
    if kind == "ragged":
        n[::2] = rng.integers(1, steps + 1, n[::2].size)
        n[1] = 0
    elif kind == "a0":
        a = rng.normal(size=(B, s.N)) + 1j * rng.normal(size=(B, s.N))
        kw["a0"] = a / np.linalg.norm(a, axis=1, keepdims=True)
        del kw["init_channel"]
    elif kind == "off":
        c0[0, 0], c0[0, 3], c0[1, 0], c0[1, 3] = s.R_grid[0] + 0.01, -20 * k[0], s.R_grid[-1] - 0.01, k[1]
    elif kind == "blowup":
        kw["dt"][1] = 1e300
    return kw


# N, K, complex, B, steps, kind, binned?
CASES = {
    "slice_real": (520, 12, False, 3, 11, "", True),
    "slice_real_64": (520, 12, False, 64, 3, "ragged", True),
    "slice_real_65": (520, 12, False, 65, 3, "", False),
    "slice_complex": (365, 12, True, 5, 11, "a0", True),
    "under_slice": (340, 12, True, 5, 5, "", False),
    "any_count": (620, 8, True, 70, 3, "off", True),
    "one": (365, 12, True, 1, 11, "", True),
    "work": (160, 64, True, 600, 4, "", False),            # below 1 GB of slices
    "work_more": (160, 64, True, 700, 4, "", True),
    "small_slice": (128, 64, True, 1100, 2, "", False),
    "work_ragged": (176, 64, True, 1100, 5, "ragged", True),
    "many_knots": (160, 1000, True, 700, 2, "", False),
    "at": (365, 12, True, 5, 11, "at", True),
    "blowup": (365, 12, True, 4, 6, "blowup", True),
    "longest": (1030, 6, False, 2, 11, "", True),
}


def both(ctx, s, sid, B, kw):
    ids, Ns = [sid] * B, [s.N] * B
    ref = ctx.run_host(ids, Ns, schedule="gemv", **kw)
    ctx.set_profiling(True)
    ctx.profile_read()
    got = ctx.run_host(ids, Ns, **kw)
    launches = ctx.profile_read()[1]
    ctx.set_profiling(False)
    return ref, got, launches


def agree(got, ref, tol=1e-10):
    for f in ("steps", "rejects", "status", "t_final"):
        assert np.array_equal(got[f], ref[f]), f
    ok = (ref["status"] & 16) == 0
    N = ref["P"].size // ok.size
    for f in ("P", "a_final"):
        d = np.abs(got[f] - ref[f]).reshape(-1, N)[ok]
        assert np.max(d) < tol, f
    d = np.abs(got["classical"] - ref["classical"]) / (1 + np.abs(ref["classical"]))
    assert np.max(d[ok]) < tol
    for f in ("norm_err", "energy_err", "angmom_err"):
        assert np.max(np.abs(got[f] - ref[f])[ok]) < 100 * tol, f


@pytest.mark.parametrize("name", list(CASES))
def test_choice_equals_per_trajectory(ctx, name):
    N, K, cplx, B, steps, kind, binned = CASES[name]
    print("[gpu] auto binned %s" % name, flush=True)
    s = system(N, K, cplx)
    sid = ctx.load_system(s, storage="C128" if cplx else "R64")
    kw = batch(s, B, steps, kind)
    if kind == "at":
        ctx.set_driver(sid, np.real(np.einsum("knn->k", s.M)) / s.N)
        kw["dynamics"] = "at"
    ref, got, launches = both(ctx, s, sid, B, kw)
    assert launches == (4 * int(np.max(kw["n_steps"])) + 1 if binned else 1)
    agree(got, ref)
    if kind == "off":
        assert ref["status"][0] & 8 and ref["classical"][1, 0] > s.R_grid[-1]
    if kind == "blowup":
        assert ref["status"][1] & 16 and not np.any(np.delete(ref["status"], 1) & 16)
    if name == "slice_real":          # in two calls, bit for bit
        ids, Ns = [sid] * B, [s.N] * B
        ctx.run_host(ids, Ns, **dict(kw, n_steps=np.array([4, 1, 7])))
        two = ctx.run_host(ids, Ns, n_steps=kw["n_steps"] - np.array([4, 1, 7]), resume=True)
        assert np.array_equal(two["a_final"], got["a_final"])
        assert np.array_equal(two["classical"], got["classical"])
    ctx.free_system(sid)


@pytest.mark.parametrize("form", ["fp32", "sparse", "mixed", "binned_off"])
def test_forms_that_stay_per_trajectory(ctx, form):
    print("[gpu] auto binned %s" % form, flush=True)
    s = system(520, 8, False)
    storage = "R32" if form == "fp32" else "R64"
    sid = ctx.load_system(s, storage=storage, layout="sparse" if form == "sparse" else "dense")
    kw = batch(s, 3, 2)
    ids = [sid] * 3
    extra = {}
    if form == "mixed":
        ids[1] = ctx.load_system(s, storage=storage)
    if form == "binned_off":
        extra["schedule"] = "gemv"
    ctx.set_profiling(True)
    ctx.profile_read()
    ctx.run_host(ids, [s.N] * 3, **extra, **kw)
    assert ctx.profile_read()[1] == 1
    ctx.set_profiling(False)
    for i in set(ids):
        ctx.free_system(i)


def test_several_passes_and_no_room(gpu_lib):
    # over 160 B x 140 columns x 60,000 trajectories: more than one pass's 1 GiB of workspace
    print("[gpu] auto binned passes", flush=True)
    ctx = gpu_lib.Context()
    s = system(140, 8, True)
    sid = ctx.load_system(s, storage="C128")
    B = 60000
    kw = batch(s, B, 2, "ragged")
    ids, Ns = [sid] * B, [s.N] * B
    ref = ctx.run_host(ids, Ns, schedule="gemv", **kw)
    os.environ["MQCT_FAULT"] = "alloc"      # no room: the per-trajectory kernels run
    try:
        got = ctx.run_host(ids, Ns, **kw)
    finally:
        del os.environ["MQCT_FAULT"]
    assert np.array_equal(got["a_final"], ref["a_final"])
    assert np.array_equal(got["classical"], ref["classical"])
    got = ctx.run_host(ids, Ns, **kw)
    assert not np.array_equal(got["a_final"], ref["a_final"])
    agree(got, ref)
    ctx.close()

"""The shared-stream form (small batches on the default schedule, work-list tails) (GPU).

The library's choice against the per-trajectory schedule's own kernel, and the work
list's forced shared-stream shape against its row-split one: sizes whose column groups
fill one thread to half the workgroup, more shares than stored rows, dense and sparse
tables, every storage type, a grid too long for LDS and a non-uniform one, J_x rows of
more than four entries, AT dynamics, paths that leave the grid at both ends, ragged step
counts with zero, and a resumed run.  The two forms differ in the order of their sums:
1e-12 of an amplitude with FP64 tables over some hundred stages, 1e-6 with FP32.
"""
import numpy as np
import pytest

from synth import systems as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    c.set_option("autotune", 0)
    yield c
    c.set_option("autotune", 1)
    c.synchronize()
    c.close()


def random_system(N, K=60, cplx=True, jw=0, log=False):
    R_ang = np.geomspace(2.0, 20.0, K) if log else None
    s = S.large_random_system(N=N, K=K, cfg_index=31, workers=0, R_ang=R_ang)
    if not cplx:
        s.M = np.ascontiguousarray(s.M.real)
    if jw:
        s.E = np.full(N, s.E[0])                       # J_x couples equal energies
        r, c = [], []
        for d in range(1, jw // 2 + 1):
            i = np.arange(N - d)
            r += [i, i + d]
            c += [i + d, i]
        s.jx_row, s.jx_col = np.concatenate(r).astype(np.int32), np.concatenate(c).astype(np.int32)
        s.jx_val = np.full(s.jx_row.size, 0.3)
    return s


CASES = {
    "rotor9": lambda: (S.rotor_atom_system(jmax=2), "R64", "dense", {}),
    "rotor16_32": lambda: (S.rotor_atom_system(jmax=3), "R32", "sparse", {}),
    "two_rotor": lambda: (S.rotor_rotor_system(jmax=3), "R64", "sparse", {}),
    "two_rotor_32": lambda: (S.rotor_rotor_system(jmax=2), "R32", "dense", {}),
    "long_grid": lambda: (random_system(33, K=700), "C128", "dense", {}),
    "log_grid": lambda: (random_system(100, log=True), "C64", "dense", {}),
    "wide_jx": lambda: (random_system(49, cplx=False, jw=8), "R64", "dense", {}),
    "half_block": lambda: (random_system(250), "C128", "dense", {}),
    "half_block_64": lambda: (random_system(500), "C64", "dense", {}),
    "off_grid": lambda: (S.rotor_atom_system(jmax=3), "R64", "dense", {"off": True}),
    "at": lambda: (S.rotor_atom_system(jmax=4), "R64", "dense", {"at": True}),
}


def batch(s, off=False):
    rng = np.random.default_rng(3)
    B = 6
    R0 = np.array([7.0, 9.0, 12.0, 15.0, 20.0, 30.0])
    E = np.full(B, 4e-3)
    if off:                       # into the wall below the first knot, and out past the last
        R0 = np.array([4.1, 4.3, 37.5, 37.7, 4.2, 37.6])
    c0 = np.zeros((B, 6))
    c0[:, 0], c0[:, 1] = R0, 0.5 * np.pi
    k = np.sqrt(2 * s.mu * E)
    c0[:, 3] = np.where(R0 > 35, k, -k) if off else -k
    c0[:, 5] = rng.uniform(0.0, 2.0, B) * k
    if off:
        c0[:2, 3] *= 30.0
    return dict(init_channel=rng.integers(0, s.N, B).astype(np.int32), classical0=c0,
                dt=np.full(B, 15.0), n_steps=np.array([25, 0, 1, 7, 25, 12]))


@pytest.mark.parametrize("name", list(CASES))
def test_auto_small_batch_equals_per_trajectory(ctx, name):
    s, storage, layout, opt = CASES[name]()
    print("[gpu] shared %s N=%d %s %s" % (name, s.N, storage, layout), flush=True)
    sid = ctx.load_system(s, storage=storage, layout=layout)
    kw = batch(s, opt.get("off", False))
    if opt.get("at"):
        ctx.set_driver(sid, np.real(np.einsum("knn->k", s.M)) / s.N)
        kw["dynamics"] = "at"
    ids, Ns = [sid] * 6, [s.N] * 6
    ref = ctx.run_host(ids, Ns, schedule="gemv", **kw)
    tol = 1e-12 if storage in ("R64", "C128") else 1e-6
    runs = {"auto": ctx.run_host(ids, Ns, **kw)}
    for tail in (0, 2):
        ctx.set_option("tail", tail)
        runs["queue%d" % tail] = ctx.run_host(ids, Ns, schedule="queue", **kw)
    ctx.set_option("tail", 1)
    for k, g in runs.items():
        assert np.max(np.abs(g["a_final"] - ref["a_final"])) < tol, k
        d = np.abs(g["classical"] - ref["classical"]) / (1 + np.abs(ref["classical"]))
        assert np.max(d) < tol, k
        for f in ("steps", "status", "t_final"):
            assert np.array_equal(g[f], ref[f]), (k, f)
        for f in ("energy_err", "norm_err", "angmom_err"):
            assert np.max(np.abs(g[f] - ref[f])) < 10 * tol * (1 + np.max(np.abs(ref["classical"]))), (k, f)
    if opt.get("off"):
        assert np.any(ref["status"] & 8) and np.any(ref["classical"][:, 0] > s.R_grid[-1])
    # the run in two calls equals the whole run bit for bit
    if not opt:
        first = np.minimum(kw["n_steps"], 5)
        ctx.run_host(ids, Ns, **dict(kw, n_steps=first))
        two = ctx.run_host(ids, Ns, n_steps=kw["n_steps"] - first, resume=True)
        assert np.array_equal(two["a_final"], runs["auto"]["a_final"])
        assert np.array_equal(two["classical"], runs["auto"]["classical"])
    ctx.free_system(sid)


@pytest.mark.parametrize("name", ["rotor9", "two_rotor", "long_grid", "wide_jx"])
def test_adaptive_tail_shape_equals_row_split(ctx, name):
    s, storage, layout, _ = CASES[name]()
    print("[gpu] shared dp5 %s" % name, flush=True)
    sid = ctx.load_system(s, storage=storage, layout=layout)
    kw = {k: v for k, v in batch(s).items() if k in ("init_channel", "classical0")}
    out = []
    for tail in (0, 2):
        ctx.set_option("tail", tail)
        out.append(ctx.run_host([sid] * 6, [s.N] * 6, schedule="queue", integrator="dp5", rtol=1e-8,
                                atol=1e-8, max_steps=40, **kw))
    ctx.set_option("tail", 1)
    ctx.free_system(sid)
    for f in ("steps", "rejects", "status"):
        assert np.array_equal(out[0][f], out[1][f]), f
    assert np.max(np.abs(out[0]["a_final"] - out[1]["a_final"])) < 1e-7     # 10 rtol
    assert np.max(np.abs(out[0]["t_final"] / out[1]["t_final"] - 1)) < 1e-7

"""The workspace that a context keeps between calls (GPU): it is given back where another
allocation of the context finds no memory, and the calls that use it take it again with the
same results.  MQCT_FAULT=full refuses each allocation while there is workspace to give back; no
kernel is made to fail.  Whether the workspace is held is read from the route of a run whose
every allocation is refused: the binned products where it is, the per-trajectory kernel where
it is not (the count of free memory does not always follow a release at once)."""
import os

import numpy as np
import pytest

from synth import systems as S

pytestmark = pytest.mark.gpu


def refused(value, f):
    os.environ["MQCT_FAULT"] = value
    try:
        return f()
    finally:
        del os.environ["MQCT_FAULT"]


def holds_workspace(ctx, run):
    ctx.set_profiling(True)
    ctx.profile_read()
    refused("alloc", run)
    launches = ctx.profile_read()[1]
    ctx.set_profiling(False)
    assert launches in (1, 5)      # per-trajectory; one step of four stages and the end's
    return launches == 5


def test_given_back_when_memory_runs_out(gpu_lib):
    print("[gpu] workspace given back", flush=True)
    s = S.large_random_system(N=365, K=12, cfg_index=37, workers=0)
    small = S.rotor_atom_system(jmax=2)
    ctx = gpu_lib.Context()
    sid = ctx.load_system(s, storage="C128")
    B = 4000
    rng = np.random.default_rng(3)
    c0 = np.zeros((B, 6))
    c0[:, 0], c0[:, 1], c0[:, 3] = rng.uniform(6.0, 30.0, B), 0.5 * np.pi, -3.0
    kw = dict(init_channel=rng.integers(0, s.N, B).astype(np.int32), classical0=c0,
              dt=np.full(B, 8.0), n_steps=np.full(B, 1))
    run = lambda: ctx.run_host([sid] * B, [s.N] * B, **kw)
    ref = run()
    assert holds_workspace(ctx, run)
    refused("full", lambda: ctx.load_system(small))
    assert not holds_workspace(ctx, run)
    again = run()
    for f in ("P", "a_final", "classical", "t_final", "steps", "status"):
        assert np.array_equal(ref[f], again[f]), f
    # a run whose own buffers must grow gives it back and takes it again
    kw = {k: np.concatenate([v, v]) for k, v in kw.items()}
    twice = refused("full", lambda: ctx.run_host([sid] * (2 * B), [s.N] * (2 * B), **kw))
    assert np.array_equal(twice["a_final"].reshape(2, -1)[0], ref["a_final"].reshape(-1))
    assert np.array_equal(twice["a_final"].reshape(2, -1)[1], ref["a_final"].reshape(-1))
    ctx.close()

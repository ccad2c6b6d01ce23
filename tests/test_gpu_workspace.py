"""The workspace that a context keeps between calls (GPU): it is given back where another
allocation of the context finds no memory, and the calls that use it take it again with the
same results.  MQCT_FAULT=full refuses each allocation while there is workspace to give back; no
kernel is made to fail."""
import os

import numpy as np
import pytest

from synth import systems as S

pytestmark = pytest.mark.gpu


def free_bytes(torch):
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_given_back_when_memory_runs_out(gpu_lib):
    import torch
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
    sid2 = ctx.load_system(small)          # grows the system table, so the next load does not
    ctx.free_system(sid2)
    held = free_bytes(torch)
    os.environ["MQCT_FAULT"] = "full"
    try:
        sid2 = ctx.load_system(small)
    finally:
        del os.environ["MQCT_FAULT"]
    # 192 bytes a trajectory and padded channel and more: 4000 x 368 take 280 MB
    assert free_bytes(torch) - held > 200e6
    again = run()
    for f in ("P", "a_final", "classical", "t_final", "steps", "status"):
        assert np.array_equal(ref[f], again[f]), f
    # a run whose own buffers must grow gives it back and takes it again
    kw = {k: np.concatenate([v, v]) for k, v in kw.items()}
    os.environ["MQCT_FAULT"] = "full"
    try:
        twice = ctx.run_host([sid] * (2 * B), [s.N] * (2 * B), **kw)
    finally:
        del os.environ["MQCT_FAULT"]
    assert np.array_equal(twice["a_final"].reshape(2, -1)[0], ref["a_final"].reshape(-1))
    assert np.array_equal(twice["a_final"].reshape(2, -1)[1], ref["a_final"].reshape(-1))
    ctx.close()

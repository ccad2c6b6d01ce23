"""The coupling builder when it cannot go on (GPU): every allocation of a build refused in
turn leaves the caller's outputs as they were, at the return and after everything that the
context's stream holds, and the next build is whole.  Only allocation calls are refused; no
kernel is made to fail."""
import os

import numpy as np
import pytest

import oracle
from synth import coupling as C

pytestmark = pytest.mark.gpu

TERMS = [(l1, 0, l2, l) for l1 in range(3) for l2 in range(2)
         for l in range(abs(l1 - l2), l1 + l2 + 1)]


@pytest.mark.parametrize("outputs", ["M", "G", "MG"])
def test_refused_build_leaves_the_outputs_alone(gpu_lib, outputs, monkeypatch):
    import torch
    print("[gpu] coupling build refused, outputs %s" % outputs, flush=True)
    basis = C.top_rotor_basis(1, (0, 1))
    ex = C.synthetic_expansion(TERMS, np.linspace(4.0, 12.0, 5), seed=5)
    ctx = gpu_lib.Context()
    made = []

    def empty(shape, **kw):
        t = torch.full(shape, -7.5, **kw)
        made.append(t)
        return t

    kw = dict(tables="M" in outputs, angular="G" in outputs)
    monkeypatch.setattr(ctx, "torch", type("T", (), dict(empty=staticmethod(empty),
                                                       float64=torch.float64)))
    refused = 0
    for n in range(1, 16):
        made.clear()
        os.environ["MQCT_FAULT"] = "alloc@%d" % n
        try:
            out = ctx.build_couplings(basis, ex, **kw)
        except gpu_lib.MQCTError as e:
            assert e.code == gpu_lib.ERR_OOM
            refused += 1
            torch.cuda.synchronize()
            assert len(made) == len(outputs)
            assert all(bool(torch.all(t == -7.5)) for t in made)
            continue
        finally:
            del os.environ["MQCT_FAULT"]
        break
    assert refused >= 1
    M_o, G_o = oracle.coupling_tables(basis, ex)
    for k, ref in (("M", M_o), ("G", G_o)):
        if k in outputs:
            assert np.max(np.abs(out[k].cpu().numpy() - ref)) < 1e-13 * np.abs(ref).max()
    ctx.close()


def test_profile_counts_one_launch_per_build(gpu_lib):
    """The timed intervals of a build are its clearing and its fill, one launch together."""
    import torch
    print("[gpu] coupling build timed", flush=True)
    basis = C.top_rotor_basis(2, (0, 1, 2))
    ex = C.synthetic_expansion(TERMS, np.linspace(4.0, 12.0, 16), seed=5)
    ctx = gpu_lib.Context()
    ctx.build_couplings(basis, ex)
    ctx.set_profiling(True)
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    e[0].record()
    for _ in range(3):
        ctx.build_couplings(basis, ex)
    e[1].record()
    torch.cuda.synchronize()
    ms, launches, by = ctx.profile_read(with_bytes=True)
    ctx.set_profiling(False)
    ctx.close()
    assert launches == 3 and by == 3 * 16 * basis.N ** 2 * 8
    assert 0 < ms < e[0].elapsed_time(e[1])

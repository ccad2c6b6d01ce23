"""What the work list's autotuner keeps (GPU): a choice made on a small batch does not stand
for a large one, nor one made on sparse tables for dense ones, and a choice once made is
reused.  Read from the tuning report; the results of the large batch agree with those of a
context that never ran the small one to 10 x the tolerance of the adaptive steps (the two may
choose different shapes)."""
import numpy as np
import pytest

from synth import systems as S

pytestmark = pytest.mark.gpu

DP5 = dict(integrator="dp5", rtol=1e-8, atol=1e-8, max_steps=30)


def start(b, B):
    i = np.arange(B) % b.B
    return dict(init_channel=b.init_channel[i], E_coll=b.E_coll[i], b=b.b[i], R0=b.R0[i])


@pytest.mark.parametrize("method", ["dp5", "rk4"])
def test_small_batch_first(gpu_lib, method):
    import torch
    print("[gpu] tuning, small batch first, %s" % method, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    (s,), b = S.config4(n_traj=64, n_steps=8)
    large = cus + 30

    def run(ctx, sid, B):
        kw = DP5 if method == "dp5" else dict(dt=np.full(B, b.dt[0]), n_steps=np.full(B, 8),
                                              schedule="queue")
        return ctx.run_host([sid] * B, [s.N] * B, **start(b, B), **kw)

    def report(ctx):
        return [e for e in ctx.tuning_report() if e["npad"] == 256]

    ctx = gpu_lib.Context()
    sp = ctx.load_system(s, layout="sparse")
    run(ctx, sp, 5)
    assert [e["wide"] for e in report(ctx)] == [False]
    g = run(ctx, sp, large)
    rep = report(ctx)
    assert [e["wide"] for e in rep] == [False, True]
    assert all(len(e["tail_candidates"]) >= 2 for e in rep)
    assert rep[0]["block"] == rep[1]["block"] and rep[0]["candidates"] == rep[1]["candidates"]
    assert rep[0]["tail_candidates"] != rep[1]["tail_candidates"]      # timed again
    dn = ctx.load_system(s, layout="dense")
    run(ctx, dn, 5)
    rep = report(ctx)
    assert len(rep) == 3 and rep[2]["rows"] == 256 and rep[0]["rows"] < 256
    run(ctx, sp, 9), run(ctx, dn, 7), run(ctx, sp, large + 5)
    assert report(ctx) == rep
    ctx.close()
    ctx = gpu_lib.Context()
    h = run(ctx, ctx.load_system(s, layout="sparse"), large)
    ctx.close()
    assert np.array_equal(g["status"], h["status"])
    assert np.max(np.abs(g["P"] - h["P"])) < 1e-7

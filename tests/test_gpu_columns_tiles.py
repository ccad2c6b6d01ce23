"""The columns schedule at the edges of its column tiles and row chunks (GPU).

Column counts around the lane groups (8, 16, 32 lanes of two columns) and the 64-column
tile, odd ones among them, two paths of different length in one call; rows of up to 150
elements (three 64-element chunks, the last partial) and rows with the diagonal alone;
real and complex, FP64 and FP32 tables; against the oracle: FP64 to 1e-12 (the rounding
of 60 stages), FP32 to 1e-6 (products rounded to 6e-8 of a coupling angle below one).
"""
import numpy as np
import pytest

import oracle
from synth import systems as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.synchronize()
    c.close()


def system(cplx):
    s = S.large_random_system(N=150, K=40, cfg_index=21, workers=0)
    if not cplx:
        s.M = np.ascontiguousarray(s.M.real)
    keep = np.ones((150, 150), bool)
    keep[:3, :] = keep[:, :3] = False          # three channels coupled to nothing
    keep[5, 20:] = keep[20:, 5] = False        # and a short row
    np.fill_diagonal(keep, True)
    s.M = np.where(keep[None], s.M, 0.0)
    s.E = np.repeat(np.sort(s.E)[::2], 2)      # pairs of equal energy, coupled by J_x
    i = np.arange(0, 150, 2)
    s.jx_row, s.jx_col = np.concatenate([i, i + 1]).astype(np.int32), np.concatenate(
        [i + 1, i]).astype(np.int32)
    s.jx_val = np.full(150, 0.5)
    return s, keep


@pytest.mark.parametrize("storage,cols", [("R64", 1), ("R64", 17), ("R64", 33), ("R64", 65),
                                          ("R32", 2), ("R32", 16), ("R32", 64), ("R32", 127),
                                          ("C128", 31), ("C128", 66), ("C64", 15), ("C64", 128)])
def test_columns_tile_edges(ctx, storage, cols):
    s, keep = system(storage[0] == "C")
    print("[gpu] columns tiles %s x %d" % (storage, cols), flush=True)
    rows, cc = np.nonzero(keep)
    sid = ctx.load_system_coo(R_grid=s.R_grid, E=s.E, rows=rows.astype(np.int32),
                              cols=cc.astype(np.int32), values=np.ascontiguousarray(s.M[:, rows, cc]),
                              mu=s.mu, jx=(s.jx_row, s.jx_col, s.jx_val), storage=storage)
    drv = np.real(np.einsum("knn->k", s.M)) / s.N
    ctx.set_driver(sid, drv)
    B = cols + 3
    path = np.concatenate([np.zeros(cols, int), np.ones(3, int)])
    kw = dict(init_channel=(np.arange(B) * 7 % s.N).astype(np.int32), E_coll=np.array([4e-3, 2e-3])[path],
              b=np.array([1.0, 3.0])[path], R0=np.array([9.0, 8.0])[path], dt=np.full(B, 12.0),
              n_steps=np.array([15, 9])[path])
    g = ctx.run_host([sid] * B, [s.N] * B, schedule="columns", dynamics="at", **kw)
    ctx.free_system(sid)
    pick = np.unique(np.concatenate([np.arange(0, cols, max(1, cols // 5)), [cols - 1, cols, B - 1]]))
    sub = {k: v[pick] for k, v in kw.items()}
    o = oracle.OracleSystem(s, driver=drv).propagate(**sub)
    tol = 1e-12 if storage in ("R64", "C128") else 1e-6
    a = g["a_final"].reshape(B, s.N)[pick]
    assert np.max(np.abs(a - o["a_final"].reshape(a.shape))) < tol
    assert np.max(np.abs(g["P"].reshape(B, s.N)[pick] - o["P"])) < tol
    assert np.max(np.abs(g["norm_err"])) < 10 * tol
    assert np.array_equal(g["steps"], kw["n_steps"])

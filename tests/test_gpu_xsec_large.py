"""Cross sections of more trajectories than one launch of the level sums takes, and of more
than 2^31 (GPU), through the C ABI with device arrays."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def call(gpu_lib, ctx, P, b, init, lev, nl, sigma):
    code = gpu_lib.lib().mqct_cross_sections(
        ctx.h, 1, C.c_int64(P.shape[0]), P.shape[1], C.c_void_p(P.data_ptr()),
        C.c_void_p(b.data_ptr()), C.c_void_p(init.data_ptr()), lev.ctypes.data_as(C.c_void_p), nl,
        C.c_double(3.0), C.c_void_p(sigma.data_ptr()))
    ctx._check(code)


def test_several_launches(gpu_lib):
    """3 x 2^20 + 5 trajectories of two channels, sums of integers and halves: exact."""
    import torch
    print("[gpu] xsec, several launches", flush=True)
    B = 3 * (1 << 20) + 5
    ctx = gpu_lib.Context()
    i = torch.arange(B, device="cuda")
    P = torch.stack([(i % 3).double(), (i % 5).double()], 1).contiguous()
    b = torch.full((B,), 0.5, dtype=torch.float64, device="cuda")
    init = (i % 2).int()
    sigma = torch.empty((2, 2), dtype=torch.float64, device="cuda")
    call(gpu_lib, ctx, P, b, init, np.array([1, 0], np.int32), 2, sigma)
    for l in range(2):
        sel = P[init == l]
        ref = 2 * np.pi * 3.0 / sel.shape[0] * 0.5 * sel.sum(0).flip(0)
        assert torch.allclose(sigma[l], ref, rtol=1e-15, atol=0)
    ctx.close()


def test_more_than_two_to_the_31(gpu_lib):
    """One channel, one level; three trajectories of the last ones start in it, the others
    in no level (the estimator skips them)."""
    import torch
    B = (1 << 31) + 7
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 61 GB of device memory")
    print("[gpu] xsec, B = 2^31 + 7", flush=True)
    ctx = gpu_lib.Context()
    P = torch.ones((B, 1), dtype=torch.float64, device="cuda")
    b = torch.ones(B, dtype=torch.float64, device="cuda")
    init = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    for k, at in enumerate((5, (1 << 31) - 1, B - 1)):
        init[at] = 0
        P[at, 0], b[at] = k + 1.0, 2.0
    sigma = torch.zeros((1, 1), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    call(gpu_lib, ctx, P, b, init, np.zeros(1, np.int32), 1, sigma)
    ctx.close()
    assert abs(float(sigma[0, 0]) / (2 * np.pi * 3.0 / 3 * 12.0) - 1) < 1e-14
    del P, b, init
    torch.cuda.empty_cache()

"""The GEMMs on 64-row tiles against the 128-row ones, bit for bit.

Products of few tiles run on 64-row tiles by default; a forced tile width takes them to the
128-row kernels.  The accumulators are whole numbers, so Y, dX and dW must be the same bits.
The step-size gradients are fp64 sums over tiles in another order, rounded to fp32 at the
end: at most one unit in the last place apart.  Parity of the default against the oracle is
checked elsewhere; N, C and D leave partial tiles on every side, and N = 1000 takes more
stages of dW (8) than there are stage buffers.
"""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import (check_plan, dev_tensor, need_gpu, run_backward, run_forward, say, to_np, TORCH_DT)
from test_gpu_lsq import _case, _steps, run_backward_lsq, run_forward_lsq

pytestmark = pytest.mark.gpu

CASES = [(k, dt, N) for k, dt, N in zip(range(8), ["f32", "f16", "bf16"] * 3, [70, 1000, 129, 300, 1, 1000, 513, 640])]


@pytest.mark.parametrize("k,dt,N", CASES)
def test_small_tiles_match(k, dt, N):
    H = need_gpu()
    D, C = (384 if k == 7 else 320), 832
    lin, X, W, G = _case((N, D, C, k, dt, "lognormal"), seed=k)
    tX, tW, tG = (dev_tensor(a, dt) for a in (X, W, G))
    sx, sw = _steps(X, W, k)
    got = []
    for bn in (0, 128, 256):
        say(f"k={k} {dt} N={N} tile width {bn}")
        H.debug_set_gemm_tile_n(bn)
        try:
            Y, dX, dW = (torch.full(s, 7.0, device="cuda", dtype=TORCH_DT[dt]) for s in ((N, C), (N, D), (C, D)))
            saved = H.Saved.empty(N, D, C)
            H.hq_linear_fwd(tX, tW, Y, saved, k)
            H.lss_linear_bwd(tG, saved, dX, dW, D, k, 0, 3, 5)
            lsaved, lsq, lY = run_forward_lsq(H, X, W, k, dt, sx, sw)
            lX, lW, dstep = run_backward_lsq(H, G, lsaved, lsq, N, D, C, k, dt, 0, 3, 5)
            torch.cuda.synchronize()
        finally:
            H.debug_set_gemm_tile_n(0)
        got.append(([Y, dX, dW, lY, lX, lW], to_np(dstep)))
    for outs, ds in got[1:]:
        for name, a, b in zip(("Y", "dX", "dW", "lsq Y", "lsq dX", "lsq dW"), got[0][0], outs):
            assert torch.equal(a, b), name
        assert (abs(ds - got[0][1]) <= 2.0 ** -23 * abs(got[0][1])).all(), (ds, got[0][1])


@pytest.mark.parametrize("N,k", [(1, 4), (70, 0), (333, 5), (1000, 2)])
def test_small_tile_accumulators(N, k):
    """The int32 accumulators of the three products on 64-row tiles: the oracle's, and the 128-row
    kernels' (no epilogue between: a wrong sum cannot hide in a rounding)."""
    H = need_gpu()
    D, C, dt = 320, 832, "f16"
    lin, X, W, G = _case((N, D, C, k, dt, "lognormal"), seed=N)
    f = O.hq_forward(X, W, k)
    b = O.lss_backward(G, f, N, 3, 5)
    saved, Y = run_forward(H, X, W, k, dt)
    tG, plan, dX, dW = run_backward(H, G, saved, N, D, C, k, dt, N, 3, 5)
    nk = check_plan(plan, b)
    want = (f.acc, b.acc_dx, b.acc_dw)
    for bn in (0, 128, 256):
        say(f"accumulators N={N} k={k} tile width {bn}")
        H.debug_set_gemm_tile_n(bn)
        try:
            acc = [torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((N, C), (N, D), (C, D))]
            H.debug_gemm_acc(0, None, saved, acc[0], N, D, C, H.workspace(H.WS_FWD, N, D, C))
            for w in (1, 2):
                H.debug_gemm_acc(w, plan, saved, acc[w], N, D, C, H.workspace(H.WS_FROM_PLAN, N, D, C))
            torch.cuda.synchronize()
        finally:
            H.debug_set_gemm_tile_n(0)
        for name, rows, got, ref in zip(("forward", "dX", "dW"), (N, nk, C), acc, want):
            assert np.array_equal(to_np(got)[:rows], ref.astype(np.int32)), (name, bn)

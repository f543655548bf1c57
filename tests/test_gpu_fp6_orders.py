"""Row orders and operand builder of the FP6 backward at the edges of their workgroups.

The orders are made by one workgroup per 1024 tokens from counts over all of them (16 tokens a
thread, rounds of 16384); the builder packs 128 entries x 128 columns a workgroup.  With the
same sample the FP6 route's gradients equal the int8 route's bit for bit.
"""
import pytest
import torch

from gpu_util import dev_tensor, need_gpu, say, TORCH_DT
from test_gpu_lsq import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,budget_div", [("lognormal", 1), ("sparse_rows", 4)])
@pytest.mark.parametrize("N,D,C", [(1, 64, 64), (15, 128, 64), (1023, 64, 192), (1024, 192, 64), (1025, 64, 64),
                                   (2063, 320, 128), (16385, 64, 64), (49153, 64, 64), (65536, 64, 64)])
def test_fp6_orders(N, D, C, kind, budget_div):
    H = need_gpu()
    k, dt, budget = 4, "bf16", max(1, N // budget_div)
    lin, X, W, G = _case((N, D, C, k, dt, kind), seed=N)
    say(f"fp6 orders N={N} D={D} C={C} {kind}")
    tX, tW, tG = (dev_tensor(a, dt) for a in (X, W, G))
    out = []
    for fp6 in (False, True):
        Y, dX, dW = (torch.full(s, 7.0, device="cuda", dtype=TORCH_DT[dt]) for s in ((N, C), (N, D), (C, D)))
        saved = (H.saved_fp6_empty if fp6 else H.Saved.empty)(N, D, C)
        (H.hq_linear_fwd_fp6 if fp6 else H.hq_linear_fwd)(tX, tW, Y, saved, k)
        (H.lss_linear_bwd_fp6 if fp6 else H.lss_linear_bwd)(tG, saved, dX, dW, D, k, budget, 11, 2)
        torch.cuda.synchronize()
        out.append((Y, dX, dW))
    for name, a, b in zip(("Y", "dX", "dW"), *out):
        assert torch.equal(a, b), name

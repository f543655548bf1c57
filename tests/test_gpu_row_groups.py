"""Row geometry of the quantisers and sizes of the sampler, against the oracle.

Few rows and widths with odd factors take row groups wider than the row's largest power-of-two
divisor, up to a whole workgroup per row, and leave lanes idle at the row's end; the maxima
run over the tensor as one array of chunks.  Codes, row sums, deltas and the sample are bit
for bit, outputs as in the other parity tests.
"""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import (check_backward_acc, check_float_output, check_forward, check_plan, need_gpu, run_backward, run_forward,
                      say, TORCH_DT)
from test_gpu_lsq import _case, _steps, check_forward_codes, run_forward_lsq
from test_gpu_variants import _check_choice

pytestmark = pytest.mark.gpu

# (N, D, C, log2_block, dtype, grad kind): chunks per row 52 / 84 (a wave per row, the last
# lanes idle), 260 / 688 / 256 (two to eight waves per row), 129 x 4 (odd), 12 and 132; 80 chunks in blocks of 8 lanes,
# whose idle lanes must still load whole blocks
SHAPES = [
    (5, 832, 1344, 6, "f32", "lognormal"),
    (3, 4160, 11008, 5, "f16", "lognormal"),
    (16, 1024, 4096, 7, "f16", "pareto"),
    (11, 1280, 384, 7, "f16", "lognormal"),
    (37, 8256, 192, 4, "bf16", "lognormal"),
    (700, 192, 2112, 6, "bf16", "sparse_rows"),
]
IDS = [f"N{s[0]}_D{s[1]}_C{s[2]}_{s[4]}" for s in SHAPES]


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_row_groups(shape):
    H = need_gpu()
    lin, X, W, G = _case(shape, seed=5)
    N, D, C, k, dt = lin.N, lin.D, lin.C, lin.log2_block, lin.dtype
    say(f"row groups {shape}")
    f = O.hq_forward(X, W, k)
    saved, Y = run_forward(H, X, W, k, dt)
    check_forward(H, X, W, k, dt, saved, Y, f)
    budget = max(1, N // 2)
    b = O.lss_backward(G, f, budget, 9, 3)
    _, plan, dX, dW = run_backward(H, G, saved, N, D, C, k, dt, budget, 9, 3)
    check_plan(plan, b)
    check_backward_acc(H, plan, saved, b, N, D, C)
    check_float_output("dX", dX, b.dX, dt)
    check_float_output("dW", dW, b.dW, dt)
    sx, sw = _steps(X, W, k)
    saved, lsq, Y = run_forward_lsq(H, X, W, k, dt, sx, sw)
    f = O.lsq_forward(X, W, k, sx, sw)
    check_forward_codes(saved, lsq, f)
    check_float_output("Y", Y, f.Y, dt)
    _check_choice(H, X, W, dt, 7)


# one wave holding every token (N <= 512), its edges and one past; the 256-thread sampler's
# two token groups and its end (N <= 4096)
@pytest.mark.parametrize("N", [8, 511, 512, 513, 2048, 2049, 4096, 4097, 8193])
@pytest.mark.parametrize("budget", [1, 3, 4])
def test_sampler_sizes(N, budget):
    """budget 1: a single row; 3: a third of the tokens; 4: all but one of the rows that are
    not zero (the last rounds clamp one row at a time)."""
    H = need_gpu()
    lin, X, W, G = _case((N, 64, 64, 2, "f16", "lognormal"), seed=N)
    f = O.hq_forward(X, W, 2, compute_output=False)
    if budget == 4:
        bs = O.bit_split(G, 4, 1)
        nz = O.leverage_scores((bs.q_up.astype(np.int64) ** 2).sum(1), (bs.q_dn.astype(np.int64) ** 2).sum(1), f.x_sumsq)
        budget = max(1, int((nz > 0).sum()) - 1)
    elif budget == 3:
        budget = max(1, N // 3)
    say(f"sampler N={N} budget={budget}")
    saved, _ = run_forward(H, X, W, 2, "f16")
    b = O.lss_backward(G, f, budget, 4, 1)
    _, plan, _, _ = run_backward(H, G, saved, N, 64, 64, 2, "f16", budget, 4, 1)
    check_plan(plan, b)


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("N,D,C,k", [(9, 2048, 64, 5), (8200, 2048, 64, 7), (16400, 1024, 64, 5), (16385, 768, 3072, 5),
                                     (700, 4096, 11008, 7), (4099, 1088, 8192, 6), (130, 11008, 64, 5)])
def test_maximum_sees_every_place(N, D, C, k, dt):
    """One value in a tensor of zeros is its own maximum wherever it sits: the first and last rows,
    columns and lanes, rows of the second round, either tensor."""
    H = need_gpu()
    say(f"maximum {N}x{D} {C}x{D} k={k} {dt}")
    X, W = (torch.zeros(r, D, device="cuda", dtype=TORCH_DT[dt]) for r in (N, C))
    saved = H.Saved.empty(N, D, C)
    ws = H.workspace(H.WS_FWD, N, D, C)
    Y = torch.empty(N, C, device="cuda", dtype=TORCH_DT[dt])
    rng = np.random.default_rng(N + D)
    for i, T in enumerate((X, W)):
        rows = T.shape[0]
        at = {(0, 0), (rows - 1, D - 1), (rows - 1, 0), (0, D - 1), (rows // 2, D // 2 + 31)}
        at |= {(min(rows - 1, q), int(rng.integers(D))) for q in (7, 8, 511, 4095, 8127, 8128, 8191, 8192)}
        for n, (r, c) in enumerate(sorted(at)):
            T[r, c] = 1.0 + n
            H.hq_linear_fwd(X, W, Y, saved, k, ws)
            assert saved.amax.cpu()[i].item() == 1.0 + n, (i, r, c)
            T[r, c] = 0.0

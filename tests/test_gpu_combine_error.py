"""The segment sums of split rows are added in pairs: a row whose first segment
sums to 1 and every other to just under half a unit in the last place of 1, which
an addition one after another loses altogether."""
import numpy as np
import pytest

import synth
from gpu_util import build, gamma, say, spmv_gpu

pytestmark = pytest.mark.gpu

W = 1 << 18


def matrix(C, seg):
    """C equal rows of W entries: 1, then values of which `seg` sum to 0.9 * 2^-25."""
    v = np.float64(np.float32(0.9 * 2.0 ** -25 / seg))
    val = np.full((C, W), v)
    val[:, 0] = 1.0
    col = np.tile(np.arange(W, dtype=np.int32), C)
    return synth.CRS(C, W, np.arange(C + 1, dtype=np.int64) * W, col, val.reshape(-1)), 1.0 + (W - 1) * v


def bound(steps, T, nseg, groups):
    """Roundings of a term: its lane's steps, the lanes of its row in pairs, its
    group's segments sixteen at a time in pairs, the groups in pairs, the result."""
    per = -(-nseg // groups)
    return gamma(steps + T.bit_length() - 1 + 4 + -(-per // 16) + groups.bit_length() - 1 + 1, 2.0 ** -24)


@pytest.mark.parametrize("C", [1, 2, 4, 8, 16, 32, 64])
def test_single_product(C):
    T = 64 // C
    seg = max(8 * T, 32)  # a small matrix's segments: one round of loads
    A, y = matrix(C, seg)
    h = build(A, C, 1, val_dtype="f32", acc_dtype="f32", vec=1, xwindow=-1)
    assert h.info["nsplit"] == 1 and h.info["lanes_per_row"] == T
    err = np.max(np.abs(spmv_gpu(h, np.ones(W)) - y)) / y
    b = bound(seg // T, T, W // seg, 512 // C)
    say("combine C", C, "error", err, "bound", b)
    assert err <= b


@pytest.mark.parametrize("C", [8, 16, 32, 64, 128])
def test_batch(C):
    import torch
    from paper_1307_6209_amd import sellcs
    rows = min(C, 64)
    T = 64 // rows
    seg = 64 * T
    A, y = matrix(C, seg)
    hs = [build(A, C, 1, val_dtype="f32", acc_dtype="f32", xwindow=-1) for _ in range(2)]
    b = sellcs.sell_batch_create(hs)
    ys = [torch.empty(C, dtype=torch.float32, device="cuda") for _ in hs]
    x = torch.ones(W, dtype=torch.float32, device="cuda")
    sellcs.sell_batch_spmv(b, [x, x], ys)
    torch.cuda.synchronize()
    lim = bound(seg // T, T, W // seg, 1)
    for v in ys:
        err = float((v.double() - y).abs().max()) / y
        say("batch combine C", C, "error", err, "bound", lim)
        assert err <= lim

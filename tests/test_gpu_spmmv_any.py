"""The one-pass block kernel for widths that no power of two fits: the same
products in the same order as the pass kernel (chosen by ktile), so the same
bits, and within the oracle's bound."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build, say

pytestmark = pytest.mark.gpu


def product(h, X, skew):
    """Y = A X with X and Y starting `skew` doubles past an aligned address;
    the doubles around Y must stay as they were."""
    import torch
    from paper_1307_6209_amd import sellcs
    n, k = h.info["nrows"], X.shape[1]
    xb = torch.zeros(X.size + skew, dtype=torch.float64, device="cuda")
    xb[skew:] = torch.from_numpy(np.ascontiguousarray(X).reshape(-1)).cuda()
    yb = torch.full((n * k + skew + 2,), -7.0, dtype=torch.float64, device="cuda")
    yb[skew:skew + n * k] = float("nan")
    sellcs.sell_spmmv(h, xb[skew:].view(-1, k), yb[skew:skew + n * k].view(-1, k))
    torch.cuda.synchronize()
    y = yb.cpu().numpy()
    assert np.all(y[:skew] == -7.0) and np.all(y[skew + n * k:] == -7.0)
    return y[skew:skew + n * k].reshape(n, k)


@pytest.mark.parametrize("k", [3, 5, 6, 7, 9, 12, 15, 20, 24, 31, 33, 40, 63])
@pytest.mark.parametrize("C,sigma,seg", [(8, 1, 64), (16, 4000, -1), (32, 256, 64), (64, 1, -1), (128, 4000, 64)])
def test_any_width_equals_pass_kernel(k, C, sigma, seg):
    A = synth.powerlaw(4_001, seed=81)
    X = synth.block_vector(A.ncols, k, seed=82)
    h = build(A, C, sigma, seg_cols=seg, kmax=64)
    ref = build(A, C, sigma, seg_cols=seg, kmax=64, ktile=64 // min(C, 64))
    say("any width k", k, "C", C, "nsplit", h.info["nsplit"])
    Y = product(h, X, 0)
    Yh, aY = oracle.crs_spmmv_hi(A, X)
    assert np.all(np.abs(Y - Yh) <= 1e-13 * aY)
    assert np.array_equal(Y, product(ref, X, 0))


@pytest.mark.parametrize("k", [5, 16, 32, 64])
def test_any_width_from_an_odd_address(k):
    """X and Y eight bytes past a 16-byte boundary; a layout with x windows
    (two lanes per row at k = 5) and one without."""
    for A, C, xw in ((synth.stencil27(13), 32, 1), (synth.powerlaw(3_000, seed=83), 64, -1)):
        X = synth.block_vector(A.ncols, k, seed=84)
        h = build(A, C, 1, seg_cols=-1, kmax=64, xwindow=xw)
        ref = build(A, C, 1, seg_cols=-1, kmax=64, ktile=64 // min(C, 64))
        assert np.array_equal(product(h, X, 1), product(ref, X, 0))

"""The block form with the x windows staged in LDS: the same products in the
same order as the pass kernel (chosen by ktile), so the same bits; chunks
narrower and wider than what stays in registers, ragged last groups, empty
rows, window elements that only padding names, odd k and odd addresses."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build, say
from test_gpu_spmmv_any import product

pytestmark = pytest.mark.gpu


def band(n, width, seed):
    """Rows of a dense band of up to `width` columns, some empty."""
    lens = (synth.u64(seed, 31, n) % np.uint64(width + 1)).astype(np.int64)
    lens[::17] = 0
    lens[5::40] = width
    rpt = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    row = np.repeat(np.arange(n), lens)
    col = np.clip(row, 0, n - width - 1) + (np.arange(int(rpt[-1])) - rpt[row])
    return synth.CRS(n, n, rpt, col.astype(np.int32), synth.uniform(int(rpt[-1]), seed, 32))


# a group of a window holds at most 8,192 slots
MATRICES = {"stencil": lambda rows: synth.stencil27(13), "narrow": lambda rows: band(1999, 12, 1),
            "wide": lambda rows: band(1500, min(61, 8191 // rows), 2)}


@pytest.mark.parametrize("k", [2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 24, 31, 32])
@pytest.mark.parametrize("C,gc", [(16, 4), (32, 4), (32, 8), (64, 4)])
@pytest.mark.parametrize("name", list(MATRICES))
def test_block_window_equals_pass_kernel(name, C, gc, k):
    A = MATRICES[name](C * gc)
    X = synth.block_vector(A.ncols, k, seed=33)
    say("block window", name, "C", C, "group", gc, "k", k)
    for sigma in (1, 64):
        h = build(A, C, sigma, seg_cols=-1, kmax=64, xwindow=1, xwindow_chunks=gc)
        ref = build(A, C, sigma, seg_cols=-1, kmax=64, ktile=64 // C, xwindow=-1)
        Y = product(h, X, 0)
        Yh, aY = oracle.crs_spmmv_hi(A, X)
        assert np.all(np.abs(Y - Yh) <= 1e-13 * aY)
        assert np.array_equal(Y, product(ref, X, 0))
        assert np.array_equal(Y, product(h, X, 1))


def test_block_window_leaves_out_what_only_zeros_name():
    """Row 0 of X, which padding names, and rows that only explicit zeros name
    do not reach Y, as in the other block kernels."""
    A = band(1500, 40, 3)
    A.val[::3] = 0.0
    X = synth.block_vector(A.ncols, 8, seed=34)
    named = np.zeros(A.ncols, bool)
    named[A.col[A.val != 0.0]] = True
    X[~named] = np.inf
    if not named[0]:
        X[0] = np.nan
    h = build(A, 32, 1, seg_cols=-1, xwindow=1)
    Y = product(h, X, 0)
    X[~named] = 0.0
    Yh, aY = oracle.crs_spmmv_hi(A, X)
    assert np.all(np.abs(Y - Yh) <= 1e-13 * aY)

"""The one-pass block kernel of any width, every instance of it, on a layout large
enough that the rule sends it there: with chunks split over several units and
without. The same bits as the pass kernel."""
import numpy as np
import pytest

import synth
from gpu_util import build, say
from one_pass_rule import compile_driver, of_handle
from test_gpu_spmmv_any import product

pytestmark = pytest.mark.gpu


def matrix():
    """16,000 rows of 40 to 64 distinct columns, some of up to 200, some empty."""
    n, ncols = 16_000, 6_000
    lens = (40 + synth.u64(91, 1, n) % np.uint64(25)).astype(np.int64)
    lens[::97] = 65 + np.arange(lens[::97].size) * 7 % 136
    lens[5::411] = 0
    rpt = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    row = np.repeat(np.arange(n), lens)
    at = np.arange(int(rpt[-1])) - rpt[row]
    step = (synth.u64(91, 2, n) % np.uint64(27)).astype(np.int64) + 1
    col = (synth.u64(91, 3, n) % np.uint64(500)).astype(np.int64)[row] + at * step[row]
    return synth.CRS(n, ncols, rpt, col.astype(np.int32), synth.uniform(int(rpt[-1]), 92))


# lanes and pairs that the widths stand for, at the chunk heights that use them
KS = {8: [9, 20, 24, 33, 40, 63], 16: [5, 7, 9, 20, 24, 33, 40, 63], 32: [3, 5, 9, 12, 20, 24, 33, 40, 63],
      64: [3, 5, 9, 12, 20, 33, 40, 63], 128: [3, 5, 12, 31, 63]}


@pytest.mark.parametrize("seg", [64, -1])
@pytest.mark.parametrize("C", list(KS))
def test_one_pass_equals_pass_kernel(C, seg, tmp_path):
    A = matrix()
    sigma = A.nrows if seg < 0 else 1
    h = build(A, C, sigma, seg_cols=seg, kmax=64, xwindow=-1)
    ref = build(A, C, sigma, seg_cols=seg, kmax=64, xwindow=-1, ktile=64 // min(C, 64))
    assert (h.info["nsplit"] > 0) == (seg > 0)
    picked = of_handle(compile_driver(tmp_path), h, KS[C])
    say("any width, units: C", C, "seg", seg, [p[2:] for p in picked])
    assert seg < 0 or all(p[4] for p in picked), picked
    for k in KS[C]:
        X = synth.block_vector(A.ncols, k, seed=93)
        want = product(ref, X, 0)
        assert np.array_equal(product(h, X, 0), want) and np.array_equal(product(h, X, 1), want)

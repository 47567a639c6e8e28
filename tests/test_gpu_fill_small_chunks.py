"""The padded fill on both sides of its rule for tiles: large layouts of wide rows,
with chunks too low for a tile (C < 8: 64 columns a wave, each slot on its own) and
just high enough, against the oracle's layout bit for bit."""
import numpy as np
import pytest

import synth
from gpu_util import assert_layout_equal, build, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [1, 2, 4, 8])
def test_fill_of_low_chunks(C):
    n = 2048 * 64 // 50 * C + 7  # rows of 60 on average: above 2,048 waves of 64 columns
    lens = 40 + synth.u64(41, 21, n) % np.uint64(41)
    lens[n // 2: n // 2 + 9] = 0
    rpt = np.zeros(n + 1, np.int64)
    np.cumsum(lens.astype(np.int64), out=rpt[1:])
    nnz = int(rpt[-1])
    assert nnz // C // 64 >= 2048
    A = synth.CRS(n, 5000, rpt, (synth.u64(41, 22, nnz) % np.uint64(5000)).astype(np.int32), synth.uniform(nnz, 41, 23))
    for sigma, dtype in ((1, "f64"), (n, "bf16")):
        say("fill of low chunks, C", C, "sigma", sigma)
        assert_layout_equal(A, build(A, C, sigma, val_dtype=dtype, acc_dtype="f64"), C, sigma, dtype)

"""The padded fill at the edges of its ranges (64 chunk columns a wave), tiles
(1,024 slots) and of the rule that tells short chunks from wide ones, against
the oracle's layout bit for bit."""
import numpy as np
import pytest

import synth
from gpu_util import assert_layout_equal, build, say

pytestmark = pytest.mark.gpu


def crs_of(lens, seed):
    lens = np.asarray(lens, np.int64)
    rpt = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    nnz = int(rpt[-1])
    col = (synth.u64(seed, 21, nnz) % np.uint64(5000)).astype(np.int32)
    return synth.CRS(lens.size, 5000, rpt, col, synth.uniform(nnz, seed, 22))


LENGTHS = {
    "tile_edges": [7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 1023, 1024, 1025] * 9,
    "empty_runs": [3] + [0] * 9000 + [130] + [0] * 9000 + [1] * 700 + [0] * 300 + [65],
    "short": ([1, 2, 1, 0, 3, 1, 1, 8, 9] * 800)[:7001],
}


@pytest.mark.parametrize("C", [1, 2, 4, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("name", list(LENGTHS))
def test_fill_edges(name, C):
    A = crs_of(LENGTHS[name], 31)
    for sigma, dtype in ((1, "f64"), (A.nrows, "bf16")):
        say("fill", name, "C", C, "sigma", sigma)
        h = build(A, C, sigma, val_dtype=dtype, acc_dtype="f64")
        assert_layout_equal(A, h, C, sigma, dtype)

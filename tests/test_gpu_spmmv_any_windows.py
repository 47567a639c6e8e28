"""The one-pass block kernel of any width on layouts with x windows, where two
lanes share a row: windows that the LDS block form leaves alone (few slots per
element, short rows, large windows). The same bits as the pass kernel."""
import numpy as np
import pytest

import synth
from block_rule import compile_driver, of_handle
from gpu_util import build, say
from test_gpu_spmmv_any import product
from test_gpu_spmmv_xwindow import band

pytestmark = pytest.mark.gpu

# widths that take several passes of the pass kernel: two lanes per row up to 8
# right-hand sides (one and two pairs a lane), four and eight lanes above
KS = [3, 5, 6, 7, 9, 12, 13, 24, 31]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return compile_driver(tmp_path_factory.mktemp("rule"))


@pytest.mark.parametrize("C", [32, 64])
@pytest.mark.parametrize("name", ["lap5", "short"])
def test_two_lanes_per_row_equal_pass_kernel(name, C, driver):
    A = synth.lap5(71) if name == "lap5" else band(3001, 6, 5)
    h = build(A, C, 1, seg_cols=-1, kmax=64, xwindow=1)
    assert h.info["xwindow"] == 1 and of_handle(driver, h, KS) == [(0, 0)] * len(KS)
    ref = build(A, C, 1, seg_cols=-1, kmax=64, ktile=64 // C, xwindow=-1)
    for k in KS:
        say("any width on windows", name, "C", C, "k", k)
        X = synth.block_vector(A.ncols, k, seed=36)
        want = product(ref, X, 0)
        assert np.array_equal(product(h, X, 0), want) and np.array_equal(product(h, X, 1), want)

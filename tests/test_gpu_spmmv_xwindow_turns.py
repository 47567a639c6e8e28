"""The window block kernel where two and four turns take enough groups (C = 16):
the same bits as the pass kernel, with chunks of up to and of more columns than
stay in registers; the layouts are ones that the rule sends there."""
import numpy as np
import pytest

import synth
from block_rule import compile_driver, of_handle
from gpu_util import build, say
from test_gpu_spmmv_any import product
from test_gpu_spmmv_xwindow import band

pytestmark = pytest.mark.gpu

KS = [5, 7, 8, 9, 12]


@pytest.mark.parametrize("name", ["stencil", "wide"])
def test_turns_equal_pass_kernel(name, tmp_path):
    A = synth.stencil27(37) if name == "stencil" else band(49_300, 61, 4)
    h = build(A, 16, 1, seg_cols=-1, kmax=64)
    assert of_handle(compile_driver(tmp_path), h, KS) == [(4, 2)] * 3 + [(4, 4)] * 2
    ref = build(A, 16, 1, seg_cols=-1, kmax=64, ktile=4, xwindow=-1)
    for k in KS:
        say("block window turns", name, k)
        X = synth.block_vector(A.ncols, k, seed=35)
        want = product(ref, X, 0)
        assert np.array_equal(product(h, X, 0), want) and np.array_equal(product(h, X, 1), want)

"""Stores of permuted rows on both sides of the lines between the two forms: y of
2 MiB, a matrix of 16 MiB, an occupancy of one half; layouts with split chunks and
without, in a batch too."""
import numpy as np
import pytest

import synth
from gpu_util import build, check_fp64, say, spmv_gpu
from test_gpu_row_stores import crs_of

pytestmark = pytest.mark.gpu

ROWS = (2 << 20) // 8
CASES = {"y": [np.arange(ROWS + d) % 4 + 1 for d in (-1, 0, 1)],
         "matrix": [np.full(100_000, w) for w in (13, 14)],  # 15.6 and 16.8 MB
         "occupancy": [np.where(np.arange(300_000) % 32 == 0, w, 1) for w in (2, 3, 40)],
         "split": [np.where(np.arange(ROWS + 5) == 77, 9_000, 1 + np.arange(ROWS + 5) % 3)]}


@pytest.mark.parametrize("name", list(CASES))
def test_both_forms_of_the_store(name):
    import torch
    from paper_1307_6209_amd import sellcs
    for lens in CASES[name]:
        A = crs_of(lens, 9001, 81)
        x = synth.uniform(A.ncols, 82)
        h = build(A, 32, 64, xwindow=-1)
        say("row stores", name, A.nrows, "beta", h.info["beta"], "split", h.info["nsplit"])
        check_fp64(A, spmv_gpu(h, x), x)
        b = sellcs.sell_batch_create([h])
        y = torch.full((A.nrows,), float("nan"), dtype=torch.float64, device="cuda")
        sellcs.sell_batch_spmv(b, [torch.from_numpy(x).cuda()], [y])
        torch.cuda.synchronize()
        check_fp64(A, y.cpu().numpy(), x)

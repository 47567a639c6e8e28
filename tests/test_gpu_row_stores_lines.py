"""Stores of permuted rows on both sides of the lines between the two forms: y of
2 MiB, a matrix of 16 MiB or 32, x of 256 KiB, an occupancy of one half; layouts with
split chunks and without, in a batch too."""
import numpy as np
import pytest

import synth
from gpu_util import build, check_fp64, say, spmv_gpu
from test_gpu_row_stores import crs_of

pytestmark = pytest.mark.gpu

ROWS = (2 << 20) // 8
CASES = {"y": [np.arange(ROWS + d) % 4 + 1 for d in (-1, 0, 1)],
         "matrix": [np.full(100_000, w) for w in (13, 14, 27, 28)],  # y of 0.8 MB: 32.4 and 33.6 MB last
         "matrix of more rows": [np.full(200_000, w) for w in (6, 7)],  # y of 1.6 MB: 14.4 and 16.8 MB
         "x": [np.full(200_000, 8)] * 3,
         "occupancy": [np.where(np.arange(300_000) % 32 == 0, w, 1) for w in (2, 3, 40)],
         "split": [np.where(np.arange(ROWS + 5) == 77, 9_000, 1 + np.arange(ROWS + 5) % 3)]}


@pytest.mark.parametrize("name", list(CASES))
def test_both_forms_of_the_store(name):
    import torch
    from paper_1307_6209_amd import sellcs
    for ncols, lens in zip((32767, 32768, 32769) if name == "x" else (40_000,) * 4, CASES[name]):
        A = crs_of(lens, ncols, 81)
        x = synth.uniform(A.ncols, 82)
        h = build(A, 32, 64, xwindow=-1)
        say("row stores", name, A.nrows, "beta", h.info["beta"], "split", h.info["nsplit"])
        check_fp64(A, spmv_gpu(h, x), x)
        b = sellcs.sell_batch_create([h])
        y = torch.full((A.nrows,), float("nan"), dtype=torch.float64, device="cuda")
        sellcs.sell_batch_spmv(b, [torch.from_numpy(x).cuda()], [y])
        torch.cuda.synchronize()
        check_fp64(A, y.cpu().numpy(), x)

"""Stores of permuted rows on both sides of the size from which they stream,
and the batch's units of short chunks with every width they may have."""
import numpy as np
import pytest

import synth
from gpu_util import build, check_fp64, say, spmv_gpu

pytestmark = pytest.mark.gpu


def crs_of(lens, ncols, seed):
    lens = np.asarray(lens, np.int64)
    rpt = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    at = np.arange(int(rpt[-1])) - np.repeat(rpt[:-1], lens)  # distinct within a row
    first = np.repeat(synth.u64(seed, 71, len(lens)) % np.uint64(ncols), lens).astype(np.int64)
    col = (first + at) % ncols
    row = np.repeat(np.arange(len(lens)), lens)
    col = col[np.lexsort((col, row))]
    return synth.CRS(len(lens), ncols, rpt, col.astype(np.int32), synth.uniform(int(rpt[-1]), seed, 72))


@pytest.mark.parametrize("extra", [-1, 0, 1, 33])
def test_permuted_rows(extra):
    """FP64 sums of 8 MiB and a row fewer or more; one to five entries a row:
    single chunks and groups of short ones."""
    n = (8 << 20) // 8 + extra
    A = crs_of(np.arange(n) * 7 % 5 + 1, 5000, 73)
    x = synth.uniform(A.ncols, 74)
    h = build(A, 32, 4096)
    say("rows", n)
    check_fp64(A, spmv_gpu(h, x), x)


@pytest.mark.parametrize("C", [8, 16, 32, 64, 128])
def test_batch_units(C):
    """Chunks of every width up to 64 / C and one more, alone and in groups, an
    empty one and a split one among them: the batch's sums are the single
    product's with one slot per lane, bit for bit where nothing is split."""
    import torch

    from paper_1307_6209_amd import sellcs

    widths = list(range(10)) + [1] * 9 + [8, 0, 0, 2, 2, 1, 1] * 3
    mats = [crs_of(np.repeat(widths, C)[: len(widths) * C - 3], 3000, 75),
            crs_of([2500] + [1] * (3 * C) + [700, 0, 5], 3000, 76)]
    hs = [build(A, C, s, vec=1) for A in mats for s in (1, A.nrows)]
    xs = [synth.uniform(3000, 77 + b) for b in range(len(hs))]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    yd = [torch.full((h.info["nrows"],), float("nan"), dtype=torch.float64, device="cuda") for h in hs]
    batch = sellcs.sell_batch_create(hs)
    sellcs.sell_batch_spmv(batch, sellcs.BatchVectors(batch, xd, yd))
    torch.cuda.synchronize()
    for b, h in enumerate(hs):
        say("batch C", C, "matrix", b)
        y = yd[b].cpu().numpy()
        check_fp64(mats[b // 2], y, xs[b])
        if b < 2:
            assert np.array_equal(y, spmv_gpu(h, xs[b]))

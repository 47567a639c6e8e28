"""The single-vector product's own segments on split layouts: fine cuts,
their combining by several thread groups per slice, and the placement by
columns where x exceeds an L2."""
import numpy as np
import pytest

import synth
from gpu_util import build, chain_per_row, check_fp64, check_reduced, say, spmv_gpu

pytestmark = pytest.mark.gpu


def lengths_crs(lens, ncols, seed):
    """Rows of the given lengths, sorted distinct columns."""
    rng = np.random.default_rng(seed)
    rpt = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    col = np.concatenate([np.sort(rng.choice(ncols, n, replace=False)) for n in lens] + [np.empty(0)])
    return synth.CRS(len(lens), ncols, rpt, col.astype(np.int32), synth.uniform(int(rpt[-1]), seed, 18))


@pytest.mark.parametrize("C", [1, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("longest", [600, 9000])
def test_segment_counts(C, longest):
    """Chunks of 1 to `longest` columns around the cuts of the segments, and
    rows 0, 1 and 33 of every slice among them."""
    lens = [longest, 0, 33, 32, 31, 64, 65, 1, 257, 0, 511, 513] * 12 + [longest - 1]
    A = lengths_crs(lens, 20_000, 91)
    x = synth.uniform(A.ncols, 92)
    for sigma in (1, A.nrows):
        h = build(A, C, sigma)
        assert h.info["nsplit"] > 0 or longest < h.info["seg_cols"]
        say("segments C", C, "sigma", sigma, "split", h.info["nsplit"])
        y = spmv_gpu(h, x)
        check_fp64(A, y, x, m=chain_per_row(A, h, C))
        assert np.array_equal(spmv_gpu(h, x), y)


@pytest.mark.parametrize("C", [16, 32, 64])
def test_segments_placed_by_column(C):
    """x of 5.6 MB: the segments are dealt to the XCDs by their columns."""
    A = synth.rail_like(nrows=301, ncols=700_001, mean_len=900, seed=93)
    x = synth.uniform(A.ncols, 94)
    h = build(A, C, A.nrows)
    assert h.info["nsplit"] > 0
    check_fp64(A, spmv_gpu(h, x), x, m=chain_per_row(A, h, C))
    h = build(A, C, A.nrows, val_dtype="bf16", acc_dtype="f64")
    check_reduced(A, h, x, "bf16", "f64", C)


@pytest.mark.parametrize("C", [16, 32, 64, 128])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 8, 9])
def test_thin_segments(C, m):
    """Slices of which m rows, anywhere in them, are long: the columns past the
    other rows' ends are taken by the long rows alone where those are few. Widths
    around the cuts of 32, 64 and 128 columns; at C = 128 one half of a chunk
    without long rows."""
    tails = [33, 64, 65, 96, 97, 128, 129, 161, 400, 3000, 9001]
    lens = []
    for c, w in enumerate(tails):
        part = np.full(C, 1 + c % 3)
        at = (synth.u64(C + c, 61, C) % np.uint64(min(C, 64))).astype(np.int64)
        for q, r in enumerate(dict.fromkeys(at.tolist())):
            if q < m:
                part[r] = max(2, w - 37 * q)
        lens += part.tolist()
    A = lengths_crs(lens, 20_000, 95)
    x = synth.uniform(A.ncols, 96)
    for sigma in (1, A.nrows):
        h = build(A, C, sigma)
        assert h.info["nsplit"] > 0
        say("thin C", C, "rows", m, "sigma", sigma)
        check_fp64(A, spmv_gpu(h, x), x, m=chain_per_row(A, h, C))
        if C <= 64:
            r = build(A, C, sigma, row_lengths=True)
            assert np.array_equal(spmv_gpu(r, x), spmv_gpu(h, x))
    h = build(A, C, 1, seg_cols=64, val_dtype="f32", acc_dtype="f32")
    check_reduced(A, h, x, "f32", "f32", C)


@pytest.mark.parametrize("C", [16, 64, 128])
def test_thin_segments_without_copies(C):
    """Where no memory is left for the thin segments' copies the product takes
    the slots from their places: the same sums in the same order."""
    from paper_1307_6209_amd import sellcs
    lens = [3] * (4 * C)
    lens[5], lens[C + 1], lens[C + 9], lens[3 * C] = 1000, 65, 33, 300
    A = lengths_crs(lens, 5000, 97)
    x = synth.uniform(A.ncols, 98)
    full = build(A, C, 1)
    ref = spmv_gpu(full, x)
    check_fp64(A, ref, x, m=chain_per_row(A, full, C))
    for n in range(64):  # the first build that fails nowhere else
        try:
            h = build(A, C, 1, xwindow=-1, allocator=sellcs.TorchAllocator(fail_after=n))
        except sellcs.SellError:
            continue
        break
    assert h.info["device_bytes"] < full.info["device_bytes"]
    assert np.array_equal(spmv_gpu(h, x), ref)


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_batch_thin_segments(C, persistent):
    """The batch with matrices that bring thin segments, one without copies of
    them, one of a given segment width and one that is not split."""
    import torch

    from gpu_util import batch_chain_per_row
    from paper_1307_6209_amd import sellcs

    mats = []
    for b in range(6):
        lens = [1 + b % 3] * (5 * C + 3 * b)
        for r, w in enumerate([40, 33, 0, 97, 300, 65, 5000, 129, 34, 64, 45, 2]):
            lens[(r * (7 + 5 * b)) % len(lens)] = w if b != 3 else 5
        mats.append(lengths_crs(lens, 6000 + b, 101 + b))
    hs = [build(A, C, s) for A, s in zip(mats[:4], (1, 64, mats[2].nrows, 1))]
    hs.append(build(mats[4], C, 1, seg_cols=128))
    for n in range(64):
        try:
            hs.append(build(mats[5], C, 1, xwindow=-1, allocator=sellcs.TorchAllocator(fail_after=n)))
        except sellcs.SellError:
            continue
        break
    make = sellcs.sell_batch_create_persistent if persistent else sellcs.sell_batch_create
    xs = [synth.uniform(A.ncols, 111 + b) for b, A in enumerate(mats)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    yd = [torch.full((A.nrows,), float("nan"), dtype=torch.float64, device="cuda") for A in mats]
    b = make(hs)
    sellcs.sell_batch_spmv(b, sellcs.BatchVectors(b, xd, yd))
    torch.cuda.synchronize()
    for A, h, x, y in zip(mats, hs, xs, yd):
        say("batch thin C", C, "rows", A.nrows)
        check_fp64(A, y.cpu().numpy(), x, m=batch_chain_per_row(A, h, C))

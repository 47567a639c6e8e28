"""The window sort where thousands of rows have 65,280 entries or more: the
stable order by all bytes of the lengths, at a cost linear in their number, and
no work on lengths that malformed row pointers give."""
import time

import numpy as np
import pytest

import synth
from gpu_util import say

pytestmark = pytest.mark.gpu


def build(lens, sigma, rpt=None, nnz=None):
    import torch
    from paper_1307_6209_amd import sellcs
    if rpt is None:
        rpt = np.zeros(lens.size + 1, np.int64)
        np.cumsum(lens, out=rpt[1:])
        nnz = int(rpt[-1])
    col = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    val = torch.zeros(nnz, dtype=torch.float64, device="cuda")
    rpt = torch.from_numpy(rpt).cuda()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    h = sellcs.sell_build(rpt, col, val, 1, 1, sigma, xwindow=-1)
    return h, time.perf_counter() - t0


def stable_order(lens, sigma):
    return np.concatenate([a + np.argsort(-lens[a:a + sigma], kind="stable") for a in range(0, lens.size, sigma)])


@pytest.mark.parametrize("sigma", [9001, 4600])
@pytest.mark.parametrize("longest", [(1 << 17) + 5, (1 << 24) + 3])
def test_thousands_of_long_rows(sigma, longest):
    from paper_1307_6209_amd import sellcs
    n = 9001
    u = synth.u64(17, 61, n)
    lens = (65270 + u % np.uint64(700)).astype(np.int64)  # around 65,280 and 65,536, many ties
    lens[synth.u64(17, 62, n) % np.uint64(3) == 0] = 3
    lens[100::1500] = longest - np.arange(lens[100::1500].size) % 2
    lens[50::700] = 1 << 16
    say("long rows", int((lens >= 65280).sum()), "sigma", sigma, "longest", longest)
    h, _ = build(lens, sigma)
    perm = sellcs.sell_export(h, parts=("perm",))["perm"]
    sellcs.sell_destroy(h)
    assert np.array_equal(perm, stable_order(lens, sigma))


def test_long_rows_cost_little():
    """8,000 rows of 65,300 entries: the order costs far less than the rest of the
    construction, some 15 ms. (Counting every row against every other is 256,000
    steps of two dependent loads, a quarter of a second.)"""
    from paper_1307_6209_amd import sellcs
    lens = np.full(8000, 65300, np.int64)
    lens[::2] += 1
    t = {}
    for turn in range(3):
        for sigma in (1, 8000):
            h, t[sigma, turn] = build(lens, sigma)
            if sigma > 1 and turn == 0:
                perm = sellcs.sell_export(h, parts=("perm",))["perm"]
                assert np.array_equal(perm, stable_order(lens, sigma))
            sellcs.sell_destroy(h)
    plain, ordered = (min(t[s, q] for q in range(3)) for s in (1, 8000))
    say("long rows, ms: sigma 1", 1e3 * plain, "sigma n", 1e3 * ordered)
    assert ordered - plain < 0.05


def test_malformed_lengths_are_not_sorted():
    """Every row longer than the whole matrix: refused, without an order of them."""
    from paper_1307_6209_amd import sellcs
    n = 200_000
    t0 = time.perf_counter()
    with pytest.raises(sellcs.SellError) as e:
        build(None, n, np.arange(n + 1, dtype=np.int64) * 70_000, 16)
    assert e.value.status == sellcs.SELL_ERR_BAD_CRS
    say("malformed, ms", 1e3 * (time.perf_counter() - t0))

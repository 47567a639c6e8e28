"""The window sort by counting (sigma above 4,096) against the oracle's stable
order: digits' and tiles' edges, ties, and rows of 65,280 entries or more, which
both passes together do not tell apart."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build, say

pytestmark = pytest.mark.gpu

LONG = [65279, 65280, 65281, 65535, 65536, 65537, 70000, 131072, 65536 + 255, 65536 + 256]


def crs_of(lens, seed):
    lens = np.asarray(lens, np.int64)
    rpt = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=rpt[1:])
    nnz = int(rpt[-1])
    return synth.CRS(lens.size, 5000, rpt, (np.arange(nnz) % 5000).astype(np.int32), np.ones(nnz))


@pytest.mark.parametrize("kind", ["short", "bytes", "long"])
@pytest.mark.parametrize("n,sigma", [(4097, 4097), (8192, 4097), (12_289, 5000), (20_001, 20_001), (20_001, 8192)])
def test_counting_sort(kind, n, sigma):
    from paper_1307_6209_amd import sellcs
    u = synth.u64(n + sigma, 51, n)
    lens = (u % np.uint64({"short": 4, "bytes": 1025, "long": 7}[kind])).astype(np.int64)
    if kind == "long":
        at = (synth.u64(n, 52, 3 * len(LONG)) % np.uint64(n)).astype(np.int64)
        lens[at] = np.array(LONG * 3)  # ties among the longest
        lens[0], lens[-1] = 65280, 70000
    A = crs_of(lens, 53)
    say("sort", kind, n, sigma)
    h = build(A, 1, sigma)
    assert np.array_equal(sellcs.sell_export(h, parts=("perm",))["perm"], oracle.sell_build(A, 1, sigma)["perm"])

"""The copies of thin segments take at most 1/64 of the device's memory; past
that a matrix holds what its layout needs and its product is the same."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def crs(nrows, wide, every):
    """One entry a row, `wide` entries in each row that is a multiple of `every`; whole
    numbers, so that sums are exact in any order."""
    import torch
    lens = torch.ones(nrows, dtype=torch.int64, device="cuda")
    lens[::every] = wide
    rpt = torch.zeros(nrows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rpt[1:])
    col = (torch.arange(int(rpt[-1]), device="cuda") % 4096).to(torch.int32)
    return rpt, col, (col % 7 - 3).to(torch.float64)


@pytest.mark.parametrize("chunks,wide", [(2_000, 3_000), (4_000, 25_000)])
def test_thin_copies_are_bounded(chunks, wide):
    import torch
    from paper_1307_6209_amd import sellcs
    C = 16
    A = crs(chunks * C, wide, C)
    x = (torch.arange(4096, device="cuda") % 5 - 2).to(torch.float64)
    y = [torch.empty(chunks * C, dtype=torch.float64, device="cuda") for _ in range(2)]
    share = torch.cuda.mem_get_info()[1] // 64
    held, copies = [], 0
    for seg, out in ((0, y[0]), (-1, y[1])):
        h = sellcs.sell_build(*A, 4096, C, 1, seg_cols=seg, xwindow=-1)
        held.append(h.info["device_bytes"])
        split = h.info["nsplit"]
        if seg == 0:  # 8 slots of 12 bytes a column past the first, dense segment at least
            copies = chunks * (wide - h.info["seg_cols"]) * 8 * 12
        sellcs.sell_spmv(h, x, out)
        torch.cuda.synchronize()
        sellcs.sell_destroy(h)
        assert split == (chunks if seg == 0 else 0)
    say("thin copies", chunks, "share", share, "copies", copies, "held", held)
    more = held[0] - held[1]
    assert more > copies if copies < share else more < copies // 4
    assert torch.equal(*y)

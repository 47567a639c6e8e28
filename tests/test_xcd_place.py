"""Split segments dealt to the XCDs by the columns they read: the launch place of
each (csrc/xcd_place.h, on the host) and what the construction's kernels make of a
list of segments (plan_place, on the GPU)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
W, X = 4, 8


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("place") / "xcd_place_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "xcd_place_driver.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("n", [1, 7, 31, 32, 33, 63, 64, 1000, 6149])
def test_places(driver, n):
    """Every place once; XCD q holds the q-th part of the units, in order, and all
    XCDs as many; fewer than a workgroup for each are left at the end."""
    out = subprocess.run([driver], input="%d %d %d" % (n, W, X), capture_output=True, text=True, check=True).stdout
    place = np.array(out.split(), np.int64)
    assert np.array_equal(np.sort(place), np.arange(n))
    dealt = n // (W * X) * W * X
    assert np.array_equal(place[dealt:], np.arange(dealt, n))
    assert np.array_equal(place[:dealt] // W % X, np.arange(dealt) * X // max(dealt, 1))
    for q in range(X):
        assert np.all(np.diff(place[:dealt][q * dealt // X:(q + 1) * dealt // X]) > 0)


I32, I64, P = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p


class PlanArgs(ctypes.Structure):
    _fields_ = [("cl", P), ("nchunks", I64), ("ncells", I64), ("grp", I32), ("wpc", I32), ("rpw", I32), ("T", I32),
                ("cus", I32), ("seg_cols", I32), ("few", P), ("len", P), ("perm", P), ("nrows", I64), ("blocks", P),
                ("next_thin", P), ("sizes", P)]


class PlanSizes(ctypes.Structure):
    _fields_ = [("total_steps", I64), ("nsplit", I64), ("nsegs", I64), ("nsplit1", I64), ("nsegs1", I64),
                ("nwhole1", I64), ("nthin1", I64), ("max_width", I32), ("pad", I32)]


class PlanOut(ctypes.Structure):
    _fields_ = [("units", P), ("splits", P), ("units1", P), ("splits1", P), ("segs", P)]


UNIT1 = np.dtype([("item", "i4"), ("nseg", "i4"), ("jb", "i4"), ("je", "i4"), ("part", "i4"), ("thin", "i4"),
                  ("rows", "u8")])
PLACE = "_ZN4sell10plan_placeERKNS_8PlanArgsEiRKNS_9PlanSizesERKNS_7PlanOutEPKlPKilPNS_7UnitColEP12ihipStream_t"


def placed(n, live, seed, C=16, ncols=1 << 20):
    """n segments of two columns, one a chunk, whose rows (`live` of each) all name one
    random column; the segments as placed and those columns."""
    import torch
    from paper_1307_6209_amd import sellcs
    rng = np.random.default_rng(seed)
    rep = rng.integers(1, ncols, n)
    col = np.zeros((n, 2, C), np.int32)
    col[:, :, :live] = rep[:, None, None]
    segs = np.zeros(n, UNIT1)
    segs["item"] = np.arange(n)
    segs["nseg"], segs["je"], segs["part"] = 1, 2, np.arange(n) * C
    dev = [torch.from_numpy(a).cuda() for a in (segs.view(np.int64), np.arange(n + 1, dtype=np.int64) * 2 * C,
                                                col.reshape(-1))]
    out = torch.full((n * 4,), -1, dtype=torch.int64, device="cuda")
    at = torch.empty(n, dtype=torch.int64, device="cuda")
    fn = getattr(sellcs.lib(), PLACE)
    fn.restype = ctypes.c_int
    fn.argtypes = [P, ctypes.c_int, P, P, P, P, I64, P, P]
    a = PlanArgs(nchunks=n, ncells=n, grp=1, wpc=1, rpw=C, T=64 // C)
    z = PlanSizes(nsegs1=n, nsplit1=n)
    o = PlanOut(units1=out.data_ptr(), segs=dev[0].data_ptr())
    torch.cuda.synchronize()
    assert fn(ctypes.byref(a), C, ctypes.byref(z), ctypes.byref(o), dev[1].data_ptr(), dev[2].data_ptr(), ncols,
              at.data_ptr(), None) == 0
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(UNIT1)
    order = np.argsort(got["item"])
    assert np.array_equal(got[order], segs)  # every segment once, unchanged
    return got["item"], rep


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 31, 32, 1000, 6149])
def test_segments_placed_by_column(n):
    ncols = 1 << 20
    item, rep = placed(n, 16, n, ncols=ncols)
    dealt = n // (W * X) * W * X
    part = np.arange(dealt) // W % X
    bins = rep[item] * 4096 // ncols  # the order is by 4,096 ranges of columns
    parts = [bins[:dealt][part == q] for q in range(X)] if dealt else []
    assert all(len(p) == dealt // X and np.all(np.diff(p) >= 0) for p in parts)
    assert all(a[-1] <= b[0] for a, b in zip(parts, parts[1:]))
    if dealt:
        assert np.all(bins[dealt:] >= parts[-1][-1])


@pytest.mark.gpu
def test_padded_segments_keep_their_order():
    """With entries in fewer than 0.4 of the rows the segments stay in chunk order."""
    assert np.array_equal(placed(1000, 6, 5)[0], np.arange(1000))
    assert not np.array_equal(placed(1000, 7, 5)[0], np.arange(1000))

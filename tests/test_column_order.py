"""The launch order of split segments by the columns they read (batch_plan.h):
every segment once, the parts of the XCDs equal, and no column of one part
above a column of the next."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("order") / "column_order_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "column_order_driver.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("n", [1, 7, 8, 31, 32, 33, 64, 1000, 6149])
def test_order_by_column(driver, n):
    W, X = 4, 8
    rep = np.random.default_rng(n).integers(0, 1_000_000 if n % 2 else 5, n)
    out = subprocess.run([driver], input="%d %d %d\n%s\n" % (n, W, X, " ".join(map(str, rep))), capture_output=True,
                         text=True, check=True).stdout
    order = np.array(out.split(), np.int64)
    assert np.array_equal(np.sort(order[order >= 0]), np.arange(n)) and order.size % (W * X) == 0
    part = np.arange(order.size) // W % X
    cols = [rep[order[(part == q) & (order >= 0)]] for q in range(X)]
    sizes = [c.size for c in cols]
    assert max(sizes) - min(sizes) <= 1
    cols = [c for c in cols if c.size]
    assert all(np.all(np.diff(c) >= 0) for c in cols)
    assert all(a[-1] <= b[0] for a, b in zip(cols, cols[1:]))

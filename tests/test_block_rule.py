"""Which kernel a block product takes on a layout with x windows: by the chunk
width, the slots per window element, the waves that the window leaves room for
and the number of groups, as measured on both sides of each line."""
import numpy as np
import pytest

from block_rule import CUS, LDS, compile_driver, turns


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return compile_driver(tmp_path_factory.mktemp("rule"))


def layout(rows, C, group, width, maxwin, runs_per_group):
    nchunks = -(-rows // C)
    groups = -(-nchunks // group)
    return (C, group, nchunks, int(nchunks * C * width), maxwin, runs_per_group, groups * runs_per_group, LDS, CUS)


# (layout, widths k that use the windows, widths that do not)
MEASURED = {
    "125-point 60^3, C 16": (layout(60**3, 16, 4, 120.3, 1541, 30), [2, 3, 4], [5, 6, 7, 8, 9, 12, 16, 32]),
    "125-point 40^3, C 16": (layout(40**3, 16, 4, 117.9, 1141, 30), [2, 4], [5, 8, 12, 16, 32]),
    "3 unknowns, 44^3, C 16": (layout(3 * 44**3, 16, 4, 78.6, 649, 9), [2, 4, 5, 8, 12], [13, 16, 31, 32]),
    "300,000 x 1,000, up to 90, C 16": (layout(300_000, 16, 4, 47.0, 1000, 1), [2, 3, 4], [5, 8, 12, 13, 16, 32]),
    "band of 128, C 16": (layout(100_000, 16, 4, 128, 191, 1), [2, 4, 5, 8, 12, 13, 16, 31, 32], [1, 33]),
    "band of 16, C 16": (layout(500_000, 16, 4, 16.0, 79, 1), [2, 8, 12, 13, 20, 28, 31], []),
    "band of 12, C 16": (layout(600_000, 16, 4, 12.0, 75, 1), [2, 8, 12, 16, 24, 32], [13, 20, 28, 31]),
    "27-point 96^3, C 16": (layout(96**3, 16, 4, 26.6, 595, 9), [2, 4, 5, 8, 12, 16, 24, 32], [13, 20, 28, 31]),
    "27-point 34^3, C 16": (layout(34**3, 16, 4, 26.1, 403, 9), [2, 4, 16], [5, 8, 9, 12]),
    "9-point 700^2, C 16": (layout(700**2, 16, 4, 9.0, 199, 3), [2, 3, 4], [5, 8, 12, 16, 32]),
    "band of 9, C 16": (layout(600_000, 16, 4, 9.0, 72, 1), [2, 4, 5, 8, 12, 16, 32], []),
    "27-point 96^3, C 32": (layout(96**3, 32, 8, 26.6, 1351, 9), [2, 3, 4, 5, 7, 8, 12], [13, 16, 32]),
    "27-point 80^3, C 32": (layout(80**3, 32, 8, 26.6, 1255, 9), [2, 4, 8, 12, 16, 24, 32], [13, 20, 28, 31]),
    "27-point 44^3, C 32": (layout(44**3, 32, 4, 26.4, 655, 9), [2, 4, 8, 12, 16, 24, 32], [31]),
    "49-point 400^2, C 32": (layout(400**2, 32, 4, 48.8, 939, 7), [2, 4, 8, 12], [13, 16, 32]),
    "9-point 700^2, C 32": (layout(700**2, 32, 8, 9.0, 775, 3), [], [2, 3, 4, 8, 12, 16, 32]),
    "band of 16, C 32": (layout(500_000, 32, 8, 16.0, 271, 1), [2, 4, 8, 12, 16, 32], [13, 20, 31]),
    "band of 64, C 32": (layout(200_000, 32, 4, 64.0, 191, 1), [2, 4, 8, 12, 13, 16, 20, 31, 32], []),
    "27-point 60^3, C 64": (layout(60**3, 64, 4, 26.6, 1135, 9), [2, 3, 4, 5, 6, 8], [7, 9, 16, 32]),
    "9-point 700^2, C 64": (layout(700**2, 64, 4, 9.0, 775, 3), [], [2, 3, 4, 5, 6, 7, 8]),
    "19-point 90^3, C 64": (layout(90**3, 64, 4, 18.8, 1311, 9), [3, 4], [2, 5, 6, 7, 8]),
    "5-point 1000^2, C 32": (layout(1000**2, 32, 8, 5.0, 768, 3), [], list(range(2, 33))),
}


@pytest.mark.parametrize("name", list(MEASURED))
def test_rule_at_the_measured_points(driver, name):
    lay, windows, other = MEASURED[name]
    for ks, want in ((windows, True), (other, False)):
        got = turns(driver, [lay + (k,) for k in ks])
        assert [(t[0] > 0) for t in got] == [want] * len(ks), (ks, got)
        for k, (kb, n) in zip(ks, got):
            if want:  # one launch column, or two of eight twice
                assert (kb, n) == ((4, 1) if k <= 4 else (4, 2) if k <= 8 else (4, 4) if k <= 12 else (8, 2))


def test_rule_stays_within_lds(driver):
    """Whatever the layout, what is staged leaves room for two workgroups on a CU."""
    rng = np.random.default_rng(7)
    rows = []
    for _ in range(4000):
        C, group = int(rng.choice([8, 16, 32, 64, 128])), int(rng.choice([4, 8]))
        width = int(rng.integers(1, 8192 // (C * group) + 2))
        maxwin = int(rng.integers(0, 4097))
        rows.append(layout(int(rng.integers(1, 1 << 21)), C, group, width, maxwin, int(rng.integers(1, 9))) +
                    (int(rng.integers(1, 70)),))
    got = turns(driver, rows)
    assert len(got) == len(rows) and any(kb for kb, _ in got)
    for r, (kb, n) in zip(rows, got):
        if kb:
            assert r[0] in (16, 32, 64) and 2 <= r[-1] <= 32 and kb * n * (2 if kb == 8 else 1) >= r[-1]
            assert 2 * (r[4] * kb * 8 + 8 * r[5]) <= LDS
            assert (kb, n) in ((4, 1), (4, 2), (4, 4), (8, 2)) and (r[0] < 64 or n <= 2 and kb == 4)

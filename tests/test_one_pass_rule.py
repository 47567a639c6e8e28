"""Block products of widths that take several passes: one pass where it was measured
to win, the passes where few long units last as long as the product."""
import pytest

from one_pass_rule import choice, compile_driver


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return compile_driver(tmp_path_factory.mktemp("rule"))


# name: (padded slots, longest unit at C = 32), {C: (widths of one pass, widths in passes)}
MEASURED = {
    "power-law 1M, sigma n": (4_300_000, 128, {16: ([5, 7, 24], []), 32: ([3, 5, 7, 12, 24], []),
                                               64: ([3, 5, 12, 24, 40], [])}),
    "power-law 500k, sigma n": (2_200_000, 128, {8: ([9], []), 32: ([3, 5, 7, 12, 24], [])}),
    "power-law 50k, sigma n": (252_000, 128, {8: ([], [20, 24, 40]), 16: ([], [10, 20, 24, 40]), 32: ([], [10])}),
    "rail 300 x 50,000": (158_000, 128, {16: ([], [10, 20, 40]), 32: ([], [10])}),
    "random 200,003": (3_900_000, 48, {16: ([5, 7, 24], []), 32: ([3, 5, 12, 24], []), 64: ([3, 5, 24], [])}),
}


@pytest.mark.parametrize("name", list(MEASURED))
def test_rule_at_the_measured_points(driver, name):
    padded, longest, by_c = MEASURED[name]
    for C, (one, several) in by_c.items():
        most = longest if "random" in name else longest * 32 // min(C, 64)
        for ks, want in ((one, 1), (several, 0)):
            got = choice(driver, [(C, k, 0, padded, most) for k in ks])
            assert all(g[1] > 1 for g in got) and [g[4] for g in got] == [want] * len(ks), (C, ks, got)


def test_widths(driver):
    """The pass kernel's width divides k; the one pass holds k with no pair to spare."""
    for C in (8, 16, 32, 64, 128):
        rows = [(C, k, local, 10**7, 10) for local in (0, 1) for k in range(2, 65)]
        for (_, k, _, _, _), (kv, passes, lanes, pairs, _) in zip(rows, choice(driver, rows)):
            assert k % kv == 0 and kv in (1, 2, 4, 8) and passes * kv * (64 // min(C, 64)) >= k
            assert 2 * lanes * pairs >= k > 2 * lanes * (pairs - 1) and (lanes, pairs) in (
                (2, 1), (2, 2), (4, 1), (4, 2), (8, 1), (8, 2), (8, 3), (8, 4))
    assert choice(driver, [(8, 2**31 - 1, 0, 1, 1)])[0][0] == 1

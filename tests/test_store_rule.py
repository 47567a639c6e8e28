"""Which way permuted rows of y are stored, at the measured points and at the edges
of the lines between both."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MB = 1 << 20


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rule") / "store_rule_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "store_rule_driver.cpp"), "-o", exe], check=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]
    return ask


# rows, columns, entries, occupancy: through the L2 in FP64, FP32, BF16 / FP64 (None: even)
MEASURED = {
    "50,000 of up to 48": (50_000, 50_000, 1_225_000, 0.98, (1, 1, 1)),
    "120,000 of up to 40": (120_000, 120_000, 2_460_000, 0.99, (1, 1, 1)),
    "93,714 x 2,580": (93_714, 2_580, 2_437_000, 0.87, (1, 1, 1)),
    "200,003 x 20,000": (200_003, 20_000, 4_900_000, 0.99, (1, 1, 1)),
    "200,003 of up to 48": (200_003, 200_003, 4_900_000, 0.98, (0, 0, 0)),
    "200,003 of up to 12": (200_003, 200_003, 1_300_000, 1.0, (1, 1, 1)),
    "power-law 500k, sigma n": (500_000, 500_000, 2_135_000, 0.96, (0, None, 0)),
    "power-law 500k, sigma 1024": (500_000, 500_000, 2_135_000, 0.14, (1, 1, None)),
    "power-law 2M, sigma 2^14": (2_000_000, 2_000_000, 8_420_000, 0.36, (0, None, None)),
}


@pytest.mark.parametrize("name", list(MEASURED))
def test_rule_at_the_measured_points(rule, name):
    n, m, nnz, beta, want = MEASURED[name]
    got = rule([(n, a, m, a, int(nnz / beta), v, beta) for a, v in ((8, 8), (4, 4), (8, 2))])
    assert all(w is None or g == w for g, w in zip(got, want)), got


def test_edges(rule):
    y1, y2, y8 = MB // 8, 2 * MB // 8, 8 * MB // 8  # rows of FP64
    big = 10 * MB  # columns
    rows = [(y1, big, 32 * MB // 12, 1, 1), (y1 + 1, big, 32 * MB // 12, 1, 0), (y1, big, 32 * MB // 12 + 1, 1, 0),
            (y2, big, 16 * MB // 12, 1, 1), (y2 + 1, big, 1, 1, 0), (y2, big, 16 * MB // 12 + 1, 1, 0),
            (y2, MB // 32, 10**9, 1, 1), (y2, MB // 32 + 1, 10**9, 1, 0), (y2 + 1, 1, 10**9, 1, 0),
            (y8, big, 10**9, 0.49, 1), (y8 + 1, big, 10**9, 0.49, 0), (y8, big, 10**9, 0.5, 0),
            (2**31 - 1, 2**31 - 1, 2**40, 0.1, 0)]
    assert rule([(n, 8, m, 8, p, 8, b) for n, m, p, b, _ in rows]) == [w for *_, w in rows]

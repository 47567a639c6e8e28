"""The one-pass window construction at its limits (64 runs, 131,072 columns
of span, the words' and threads' shares of the bitmap), where the two-pass one
takes over beyond them: the exported tables equal the plain definition."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build, say
from xwindow_def import window_tables

pytestmark = pytest.mark.gpu


def matrix(columns, ncols, rows=203):
    """Rows 0 and 101 hold the given columns, the others one entry each."""
    columns = np.unique(np.asarray(columns, np.int64))
    out = [columns if i in (0, 101) else columns[i % columns.size:][:1] for i in range(rows)]
    rpt = np.zeros(rows + 1, np.int64)
    np.cumsum([c.size for c in out], out=rpt[1:])
    return synth.CRS(rows, ncols, rpt, np.concatenate(out).astype(np.int32), synth.uniform(int(rpt[-1]), 5, 6))


CASES = {
    "runs_64": np.arange(5, 5 + 3 * 63, 3),        # with column 0 of the padding: 64 runs
    "runs_65": np.arange(5, 5 + 3 * 64, 3),
    "span_below": [7, 7 + 131_071],
    "span_over": [7, 7 + 131_072],
    "from_one": [1, 2, 3, 131_071],                # column 0 joins the first run
    "words": np.concatenate([np.arange(31, 66), np.arange(255, 258), [511, 512, 4095, 4096]]),
    "zero_only": [0],
    "wide_run": np.arange(1000, 1250),
}


@pytest.mark.parametrize("gc", [4, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_tables_at_the_limits(name, gc):
    from paper_1307_6209_amd import sellcs
    A = matrix(CASES[name], 140_000)
    for C in (8, 16):
        say("one-pass window", name, "C", C, "group", gc)
        h = build(A, C, 1, xwindow=1, xwindow_chunks=gc, seg_cols=-1)
        lay = oracle.sell_build(A, C, 1)
        segoff, seg, lcol = window_tables(lay["col"], lay["cs"], gc)
        got = sellcs.sell_export_xwindow(h)
        assert np.array_equal(got["segoff"], segoff) and np.array_equal(got["seg"], seg)
        assert np.array_equal(got["lcol"], lcol)

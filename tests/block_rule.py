"""The block form's rule (csrc/block_rule.h), compiled for the host: which
(right-hand sides at a time, turns) a width runs with on a layout with x windows,
(0, 0) where it takes the kernels without them."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS, CUS = 160 << 10, 256  # of a compute unit; compute units


def compile_driver(folder):
    exe = str(folder / "block_rule_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "block_rule_driver.cpp"), "-o", exe], check=True)
    return exe


def turns(exe, rows):
    text = "\n".join(" ".join(map(str, r)) for r in rows)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def of_handle(exe, h, ks):
    from paper_1307_6209_amd import sellcs
    i = h.info
    runs = np.diff(sellcs.sell_export_xwindow(h)["segoff"])
    return turns(exe, [(i["C"], i["xwindow_group_chunks"], i["nchunks"], i["padded"], i["xwindow_max"],
                        int(runs.max()), i["xsegments"], LDS, CUS, k) for k in ks])

"""The choice between one pass of any width and the pass kernel (csrc/block_rule.h),
compiled for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compile_driver(folder):
    exe = str(folder / "one_pass_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "one_pass_driver.cpp"), "-o", exe], check=True)
    return exe


def choice(exe, rows):
    """(kv, passes, lanes, pairs, one pass wins) for each (C, k, local, padded, longest)."""
    text = "\n".join(" ".join(str(int(v)) for v in r) for r in rows)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def of_handle(exe, h, ks):
    i = h.info
    longest = min(i["max_row_len"], i["seg_cols"]) if i["nsplit"] else i["max_row_len"]
    return choice(exe, [(i["C"], k, i["xwindow"], i["padded"], longest) for k in ks])

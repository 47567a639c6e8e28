"""Sizes of the blocks that the block cache hands out (csrc/block_cache.h):
reported as they are, the same whatever was kept."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sizes_follow_from_the_request(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I",
                    os.path.join(ROOT, "paper_1307_6209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "block_cache_size_driver.cpp"), "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0 and p.stdout.strip() == "ok", p.stdout

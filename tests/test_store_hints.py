"""The store of a row of y keeps its two forms in the compiled kernel: streamed
past the L2 and through it. (Two stores to one address that differ in the hint only
are joined by the compiler, and then neither streams.)"""
import os
import re
import subprocess

from paper_1307_6209_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_streaming_store_survives(tmp_path):
    out = str(tmp_path / "store.s")
    subprocess.run([_build.HIPCC, *_build.CFLAGS, "-I", _build.CSRC, "--cuda-device-only", "-S",
                    os.path.join(HERE, "native", "store_hint.hip"), "-o", out], check=True, capture_output=True)
    body = open(out).read()
    body = body[body.index("store_row:"):body.index(".end_amdhsa_kernel")]
    stores = re.findall(r"global_store_dwordx2[^\n]*", body)
    assert any(s.split()[-1] == "nt" for s in stores) and any(s.split()[-1] != "nt" for s in stores), stores

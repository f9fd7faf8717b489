"""No GEMM launch takes more split-K slabs than its cap, whatever the cap, and every width and
depth that the callers accept (multiples of 64) is taken at every row count.

The caller works the cap out from the rows its partial-sum buffer holds, so it is any number
from 1 to 8.  tests/native/split_cap.cpp reads the choice of the library's own host code
(built with hipcc, host side only) over rows, widths, depths and caps.
"""
import os
import subprocess

import pytest
import torch

from paper_2609_34977_amd import _lib
from paper_2609_34977_amd.build import CSRC, PKG, ROOT, _hipcc


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="walks the dispatch with pointers that are no memory")
def test_no_launch_splits_past_its_cap(tmp_path):
    _lib.lib()  # built
    exe = str(tmp_path / "split_cap")
    r = subprocess.run([_hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "native", "split_cap.cpp"), "-o", exe,
                        "-L", PKG, "-lspider", f"-Wl,-rpath,{PKG}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    table = {p: tuple(int(x) for x in v) for p, *v in (line.split() for line in r.stdout.splitlines())}
    assert table.pop("refused") == (0,), "widths and depths of multiples of 64 are accepted"
    assert set(table) == {"few", "stream", "tile", "staged"}
    for path, (launches, split, over) in table.items():
        assert launches > 1000 and over == 0, table
        assert (split > 0) == (path != "few"), table

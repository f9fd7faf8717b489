"""The host dispatch of the fused Q, K, V GEMMs never refuses a launch of its own choosing.

A prefill layer asks once whether the three groups run fused and whether the queries go
apart; the launches that follow must be accepted whatever split a part of the groups would
have taken alone.  tests/native/qkv_dispatch.cpp walks row counts, query counts and widths
through the library's own host code (built with hipcc, host side only).
"""
import os
import subprocess

import pytest
import torch

from paper_2609_34977_amd import _lib
from paper_2609_34977_amd.build import CSRC, PKG, ROOT, _hipcc


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="walks the dispatch with pointers that are no memory")
def test_fused_qkv_launches_are_accepted(tmp_path):
    _lib.lib()  # built
    exe = str(tmp_path / "qkv_dispatch")
    r = subprocess.run([_hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "native", "qkv_dispatch.cpp"), "-o", exe,
                        "-L", PKG, "-lspider", f"-Wl,-rpath,{PKG}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    table = {int(d): (int(f), int(a), int(x)) for d, f, a, x in (line.split() for line in r.stdout.splitlines())}
    assert len(table) == 8
    for d, (fused, apart, refused) in table.items():
        assert refused == 0, (d, table)
        assert fused > apart
    assert table[4096][1] > 0 and table[5120][1] > 0  # both routes are walked

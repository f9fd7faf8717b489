"""No barrier of a kernel that fills LDS by DMA is passed with LDS accesses in flight.

After the barrier other waves' DMAs overwrite what was just read, so a read that has only been
issued may return the next data.  The compiler waits for a read where its value is used, and
may place that behind a barrier written in inline assembly.  Read from the disassembly of the
built library: within a basic block, LDS reads and writes issued and not waited for at an
s_barrier.
"""
import os
import re
import shutil
import subprocess

from paper_2609_34977_amd import _lib
from paper_2609_34977_amd.build import PKG, _hipcc


def _in_flight(text):
    """{kernel: [DMAs, barriers, barriers with LDS accesses in flight]}"""
    out, kernel, n = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", line)
        op = line.split()
        if m and m.group(1).startswith("_Z"):
            kernel, n = m.group(1), 0
            out[kernel] = [0, 0, 0]
        elif kernel is None or not op:
            continue
        elif m:
            n = 0  # another block: its predecessors are not followed
        elif op[0].startswith(("ds_read", "ds_write")):
            n += 1
        elif op[0].startswith("global_load_lds"):
            out[kernel][0] += 1
        elif op[0] == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", line)
            n = min(n, int(m.group(1))) if m else n
        elif op[0] == "s_barrier":
            out[kernel][1] += 1
            out[kernel][2] += n > 0
    return out


def test_the_reading_finds_a_missing_wait():
    ok = "00 <_Zk>:\n ds_read_b128 v1, v0\n s_waitcnt vmcnt(2) lgkmcnt(0)\n s_barrier\n global_load_lds_dwordx4 v1, off\n"
    assert _in_flight(ok) == {"_Zk": [1, 1, 0]}
    assert _in_flight(ok.replace(" lgkmcnt(0)", "")) == {"_Zk": [1, 1, 1]}


def test_no_lds_accesses_in_flight_at_a_barrier(tmp_path):
    _lib.lib()  # built
    objdump = os.path.join(os.path.dirname(os.path.realpath(_hipcc())), "..", "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    shutil.copy(os.path.join(PKG, "libspider.so"), tmp_path)
    subprocess.run([objdump, "--offloading", "libspider.so"], cwd=tmp_path, check=True, capture_output=True)
    found = {}
    for f in sorted(os.listdir(tmp_path)):
        if f.endswith("gfx950"):
            r = subprocess.run([objdump, "-d", "--symbolize-operands", "--no-show-raw-insn", f], cwd=tmp_path, check=True,
                               capture_output=True, text=True)
            found.update(_in_flight(r.stdout))
    dma = {k: v for k, v in found.items() if v[0]}
    for name in ("gemm_stream_kernel", "gemm_tile_kernel", "attention_wide_kernel", "rows32", "kmeans_pass_kernel"):
        assert any(name in k and v[1] for k, v in dma.items()), name
    assert not {k: v for k, v in dma.items() if v[2]}

"""The split-K partial sums of O and down stay inside the prefill's workspace where the rows
leave room for a number of slabs that is no power of two: 520 rows (7 slabs), and 420 active of
1100 (7 of the slabs of 420 rows).  The bytes behind the workspace must not change, with and
without a cache.  Bars as in test_gpu_prefill."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoder as odec
from synth import get_workload
from gpu_common import need_gpu, rel_err, log
from test_gpu_prefill import _oracle_weights, _x

GUARD = 32 << 20  # more than one slab of either case


@pytest.mark.gpu
@pytest.mark.parametrize("rows,active", [(520, 520), (1100, 420)])
def test_partial_sums_stay_in_the_workspace(rows, active):
    L = need_gpu()
    dec = dataclasses.replace(get_workload("llava15_7b").dec, L=1, d=2048, H=16, d_ff=4096)
    log(f"[split-cap] {active} of {rows} rows")
    cu = np.array([0, rows], np.int32)
    codes = np.zeros((1, rows), np.uint8)
    codes[0, :rows - active] = 3
    x, wts = _x(dec, rows, 3), _oracle_weights(dec, 1)
    W = [{k: torch.from_numpy(v).to("cuda", torch.float32 if "norm" in k else torch.bfloat16)
          for k, v in wts(0).items()}]
    cfg = L.decoder_cfg(1, dec.d, dec.H, dec.d_ff, L.BF16, dec.eps, dec.theta)
    size = L.prefill_workspace_size(cfg, 1, rows)
    buf = torch.full((size + 256 + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    h = L.prefill(cfg, W, cu, x.cuda(), codes, workspace=buf)
    first = -buf.data_ptr() % 256  # the workspace starts at the first 256-byte boundary
    assert bool((buf[first + size:] == 0x5A).all())
    kv = L.kv_cache(cfg, 1, rows, "cuda")
    assert torch.equal(L.prefill_kv(cfg, W, cu, x.cuda(), codes, kv), h)
    ref = odec.prefill(x.float().numpy(), wts, cu, codes, dec, recipe="bf16", dtype=np.float64, n_layers=1)
    e = rel_err(h[rows - active:].cpu().numpy(), ref[rows - active:])
    log(f"  max rel err {e:.2e}")
    assert e <= 2e-2
    assert torch.equal(h[:rows - active].cpu(), x[:rows - active].float())

"""The decoder at up to 256 rows at the edges of the weight-streaming GEMM's tiles: row counts
around the 64-row steps, a SwiGLU width that ends in the middle of a 48-column tile, K of four
and of five k-blocks (fewer than the ring's stages and the split), two ragged samples.  The
cache-filling prefill must return the same bits as the plain one.  Bars as in test_gpu_prefill."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoder as odec
from synth import get_workload
from gpu_common import need_gpu, rel_err, log
from test_gpu_prefill import _codes, _oracle_weights, _x


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [5, 63, 64, 65, 129, 193, 256])
def test_stream_rows_and_ragged_columns(rows):
    L = need_gpu()
    n_layers = 2
    dec = dataclasses.replace(get_workload("llava15_7b").dec, L=n_layers, d=256, H=2, d_ff=320)
    cu = np.array([0, rows // 3, rows], np.int32)
    log(f"[stream] rows={rows}")
    codes = _codes(n_layers, cu, 1, 7, 0.3, 0.3, True)
    x = _x(dec, rows, 3)
    W = [{k: torch.from_numpy(v).to("cuda", torch.float32 if "norm" in k else torch.bfloat16)
          for k, v in _oracle_weights(dec, n_layers)(l).items()} for l in range(n_layers)]
    cfg = L.decoder_cfg(n_layers, dec.d, dec.H, dec.d_ff, L.BF16, dec.eps, dec.theta)
    h = L.prefill(cfg, W, cu, x.cuda(), codes)
    kv = L.kv_cache(cfg, 2, rows, "cuda")
    assert torch.equal(L.prefill_kv(cfg, W, cu, x.cuda(), codes, kv), h)
    assert torch.count_nonzero(kv["k"][:, 0, rows // 3:]) == 0
    ref = odec.prefill(x.float().numpy(), _oracle_weights(dec, n_layers), cu, codes, dec, recipe="bf16",
                       dtype=np.float64, n_layers=n_layers)
    e = rel_err(h.cpu().numpy(), ref)
    log(f"  max rel err {e:.2e}")
    assert e <= 2e-2

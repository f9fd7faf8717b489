"""Prefill, cache and one decode step at the edges of the decoder's dispatch:

* fp32 heads that are not a multiple of four wide (prefill), heads of three and of 24 pieces
  (the lanes of a key in the decode attention are not a power of two), GEMMs whose K is no
  multiple of 4 and of 64, and the 32 x 32 tiles of many outputs;
* more than 256 rows with four to ten k-blocks (fewer than the large tile's stages are deep
  on one side, a split of them on the other), and few queries among them (in the fused launch
  at 420 rows, through split partials at 1100);
* decode steps of 6 and of 33 samples (QKV finished in the GEMM's epilogue, one and more
  row tiles) and of 260, at a width outside
  the fused epilogues' tiles (partials and decode_qkv);
* a SwiGLU width for which the streaming GEMM takes its widest column tile (288 tiles of 48
  columns would be a second wave of blocks), over one, two and all row tiles.

Bars as in test_gpu_prefill and test_gpu_decode; the cache-filling prefill must return the
same bits as the plain one.
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decode as od
from oracle import decoder as odec
from synth import get_workload
from gpu_common import need_gpu, rel_err, log
from test_gpu_prefill import _codes, _oracle_weights, _x

F, H = "tiny", "llava15_7b"
CASES = {
    # name: (workload, d, H, d_ff, cu_seqlens, n_text, p_attn, decode step)
    "fp32_dh6": (F, 36, 6, 70, [0, 10, 47], 4, 0.3, False),
    "fp32_dh12_dff70": (F, 36, 3, 70, [0, 10, 47], 4, 0.3, True),
    "fp32_dh96_530_rows": (F, 192, 2, 1376, [0, 530], 100, 0.1, True),
    "bf16_four_k_blocks_420_rows": (H, 256, 2, 384, [0, 300, 420], 20, 0.3, True),
    "bf16_few_queries_420_rows": (H, 256, 2, 384, [0, 300, 420], 20, 1.0, True),
    "bf16_few_queries_1100_rows": (H, 512, 4, 640, [0, 1100], 120, 1.0, True),
    "bf16_six_samples": (H, 256, 2, 320, list(range(0, 61, 10)), 4, 0.3, True),
    "bf16_33_samples": (H, 256, 2, 320, list(range(0, 232, 7)), 4, 0.3, True),
    "bf16_260_samples": (H, 384, 3, 320, list(range(0, 781, 3)), 2, 0.3, True),
    "bf16_wide_ffn_40_rows": (H, 256, 2, 13824, [0, 40], 8, 0.3, True),
    "bf16_wide_ffn_100_rows": (H, 256, 2, 13824, [0, 100], 8, 0.3, False),
    "bf16_wide_ffn_256_rows": (H, 256, 2, 13824, [0, 56, 256], 30, 0.1, False),
}


@pytest.mark.gpu
@pytest.mark.parametrize("case", list(CASES))
def test_edges(case):
    L = need_gpu()
    wl, d, heads, d_ff, cu, n_text, pa, step = CASES[case]
    n_layers = 2
    dec = dataclasses.replace(get_workload(wl).dec, L=n_layers, d=d, H=heads, d_ff=d_ff)
    bf16 = dec.dtype == "bf16"
    cu = np.array(cu, np.int32)
    B, rows = len(cu) - 1, int(cu[-1])
    log(f"[edges] {case} rows={rows}")
    codes = _codes(n_layers, cu, n_text, 7, pa, 0.3, True)
    x, new = _x(dec, rows, 3), _x(dec, B, 4)
    act = torch.bfloat16 if bf16 else torch.float32
    wts = _oracle_weights(dec, n_layers)
    W = [{k: torch.from_numpy(v).to("cuda", torch.float32 if "norm" in k else act)
          for k, v in wts(l).items()} for l in range(n_layers)]
    cfg = L.decoder_cfg(n_layers, d, heads, d_ff, L.BF16 if bf16 else L.F32, dec.eps, dec.theta)
    kv = L.kv_cache(cfg, B, int(max(cu[1:] - cu[:-1])) + 3, "cuda")
    h = L.prefill(cfg, W, cu, x.cuda(), codes)
    assert torch.equal(L.prefill_kv(cfg, W, cu, x.cuda(), codes, kv), h)
    lens = (cu[1:] - cu[:-1]).astype(np.int32)
    got = L.decode_step(cfg, W, lens, new.cuda(), kv)[0].cpu().numpy() if step else None
    ref_new, _ = od.decode(x.float().numpy(), wts, cu, codes,
                            [new[b:b + 1].float().numpy() for b in range(B)], dec,
                            recipe="bf16" if bf16 else "f32")
    ref = odec.prefill(x.float().numpy(), wts, cu, codes, dec, recipe="bf16" if bf16 else "f32",
                       dtype=np.float64, n_layers=n_layers)
    tol = 2e-2 if bf16 else 1e-4
    e = rel_err(h.cpu().numpy(), ref)
    es = rel_err(got, np.stack([ref_new[b][0] for b in range(B)])) if step else 0.0
    log(f"  prefill {e:.2e}, decode step {es:.2e}")
    assert e <= tol and es <= tol

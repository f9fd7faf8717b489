"""Prefill layers with few queries among many rows: the text rows alone query while every row
gives a key and a value.

* 900 rows at d = 4096 and 600 at d = 5120: Q, K and V unsplit in one launch, where K and V
  alone would be split along k;
* 2000 rows at d = 4096: the queries go to the streaming kernel, K and V to the tile kernel;
* the online controller above 256 rows, whose admissions leave the text rows as queries.

Bars as in test_gpu_prefill; with a cache the same bits.
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoder as odec
from synth import get_workload
from gpu_common import need_gpu, rel_err, log
from test_gpu_prefill import _oracle_weights, _x

CASES = {
    # name: (workload, rows, query rows)
    "7b_900_rows_64_queries": ("llava15_7b", 900, 64),
    "13b_600_rows_64_queries": ("llava15_13b", 600, 64),
    "7b_2000_rows_64_queries": ("llava15_7b", 2000, 64),
}


def _small(workload, n_layers):
    return dataclasses.replace(get_workload(workload).dec, L=n_layers, d_ff=256)


def _weights(wts, n_layers):
    return [{k: torch.from_numpy(v).to("cuda", torch.float32 if "norm" in k else torch.bfloat16)
             for k, v in wts(l).items()} for l in range(n_layers)]


@pytest.mark.gpu
@pytest.mark.parametrize("case", list(CASES))
def test_few_queries(case):
    L = need_gpu()
    wl, rows, nq = CASES[case]
    dec = _small(wl, 1)
    log(f"[qkv-dispatch] {case}")
    cu = np.array([0, rows], np.int32)
    codes = np.zeros((1, rows), np.uint8)
    codes[0, :rows - nq] = 1
    x, wts = _x(dec, rows, 3), _oracle_weights(dec, 1)
    W = _weights(wts, 1)
    cfg = L.decoder_cfg(1, dec.d, dec.H, dec.d_ff, L.BF16, dec.eps, dec.theta)
    h = L.prefill(cfg, W, cu, x.cuda(), codes)
    kv = L.kv_cache(cfg, 1, rows, "cuda")
    assert torch.equal(L.prefill_kv(cfg, W, cu, x.cuda(), codes, kv), h)
    assert bool((kv["k"][0, 0].abs().amax(1) > 0).all()) and bool((kv["v"][0, 0].abs().amax(1) > 0).all())
    ref = odec.prefill(x.float().numpy(), wts, cu, codes, dec, recipe="bf16", dtype=np.float64, n_layers=1)
    e = rel_err(h.cpu().numpy(), ref)
    eq = rel_err(h[rows - nq:].cpu().numpy(), ref[rows - nq:])
    log(f"  max rel err {e:.2e}, query rows {eq:.2e}")
    assert e <= 2e-2 and eq <= 2e-2


@pytest.mark.gpu
def test_online_admissions_leave_few_queries():
    L = need_gpu()
    rows, n_text, V = 800, 64, 1024
    dec = _small("llava15_7b", 2)
    log(f"[qkv-dispatch] online, {rows} rows")
    cu = np.array([0, rows], np.int32)
    x = _x(dec, rows, 3).cuda()
    W = _weights(_oracle_weights(dec, 2), 2)
    cfg = L.decoder_cfg(2, dec.d, dec.H, dec.d_ff, L.BF16, dec.eps, dec.theta)
    wu = _x(dec, V, 9).cuda()
    # attention is the cheaper sub-layer everywhere and the threshold admits every visual row at layer 0
    sel, target = L.slc_policy(np.array([0.1, 0.1], np.float32), np.array([10.0, 10.0], np.float32))
    h, codes, admit, _ = L.prefill_online(cfg, W, cu, x, n_text, wu, sel, target, 3.0, 1.0, -1e6)
    n_vis = rows - n_text
    assert (admit[:n_vis] == 0).all() and (codes[:, :n_vis] == 1).all() and (codes[:, n_vis:] == 0).all()
    assert torch.equal(h, L.prefill(cfg, W, cu, x, codes))

"""fp32 prefill of the longest samples the attention's LDS holds: 40960 rows, whose scores fill
it, and 40448, the last length with the query and the partial sums beside them.  Few rows query
(the rest bypass both sub-layers); the queries are compared with 64 bits at 1e-4, and a row that
both lengths hold must have the same bits."""
import dataclasses
import math

import numpy as np
import pytest
import torch

from oracle.decoder import rmsnorm, rope, silu
from synth import get_workload
from gpu_common import need_gpu, rel_err, log
from test_gpu_prefill import _oracle_weights, _x

LONGEST, BESIDE = 40960, 40448


def _reference(x, w, queries, dec):
    d, H = dec.d, dec.H
    dh = d // H
    f = {k: v.astype(np.float64) for k, v in w.items()}
    xn = rmsnorm(x, f["attn_norm"], dec.eps)
    heads = lambda t: t.reshape(-1, H, dh)
    k = rope(heads(xn @ f["wk"].T), np.arange(len(x)), dec.theta)
    v = heads(xn @ f["wv"].T)
    q = rope(heads(xn[queries] @ f["wq"].T), np.array(queries), dec.theta)
    out = np.zeros((len(queries), H, dh))
    for i, r in enumerate(queries):
        for h in range(H):
            z = k[:r + 1, h] @ q[i, h] / math.sqrt(dh)
            p = np.exp(z - z.max())
            out[i, h] = p @ v[:r + 1, h] / p.sum()
    y = x[queries] + out.reshape(len(queries), d) @ f["wo"].T
    xn = rmsnorm(y, f["ffn_norm"], dec.eps)
    return y + (silu(xn @ f["wg"].T) * (xn @ f["wu"].T)) @ f["wd"].T


@pytest.mark.gpu
@pytest.mark.parametrize("d,H", [(8, 2), (12, 2)])  # heads of 4 (16-byte pieces) and of 6 (single elements)
def test_longest_samples(d, H):
    L = need_gpu()
    dec = dataclasses.replace(get_workload("tiny").dec, L=1, d=d, H=H, d_ff=16)
    log(f"[long-f32] d={d} H={H}")
    w = _oracle_weights(dec, 1)(0)
    W = [{k: torch.from_numpy(v).to("cuda", torch.float32) for k, v in w.items()}]
    cfg = L.decoder_cfg(1, d, H, dec.d_ff, L.F32, dec.eps, dec.theta)
    x = _x(dec, LONGEST, 3)
    got = {}
    for rows in (BESIDE, LONGEST):
        queries = [0, 63, 20000, BESIDE - 1] + ([LONGEST - 2, LONGEST - 1] if rows == LONGEST else [])
        codes = np.full((1, rows), 3, np.uint8)
        codes[0, queries] = 0
        h = L.prefill(cfg, W, np.array([0, rows], np.int32), x[:rows].contiguous().cuda(), codes).cpu()
        got[rows] = h[queries]
        skipped = np.flatnonzero(codes[0])
        assert torch.equal(h[skipped], x[skipped])
        e = rel_err(got[rows].numpy(), _reference(x[:rows].double().numpy(), w, queries, dec))
        log(f"  {rows} rows: {e:.2e}")
        assert e <= 1e-4
    assert torch.equal(got[LONGEST][:4], got[BESIDE])

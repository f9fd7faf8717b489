"""Decode attention at the lines of its two ways to the scores (by rows, by keys): the number of
blocks (heads times samples) around one per CU, the keys around each limit, and heads of 8, 16,
32 and 64 vectors per row.  One decode step of one layer against 64 bits; bars as in
test_gpu_decode (2e-2 for bf16, 1e-4 for fp32)."""
import math

import numpy as np
import pytest
import torch

from gpu_common import need_gpu, log

BF, F32 = torch.bfloat16, torch.float32
EPS, THETA = 1e-5, 10000.0
CASES = [
    # dtype, heads, head size, samples, cached keys (the new token makes one more)
    (BF, 2, 128, 1, 2047), (BF, 2, 128, 1, 2048), (BF, 2, 128, 127, 2050), (BF, 2, 128, 128, 2050),
    (F32, 2, 64, 1, 2047), (F32, 2, 64, 1, 2048), (F32, 2, 64, 128, 2050),
    (F32, 8, 32, 32, 300), (F32, 8, 32, 33, 254), (F32, 8, 32, 33, 255),
    (F32, 2, 128, 129, 254), (F32, 2, 128, 129, 255), (F32, 2, 128, 3, 300),
    (F32, 1, 256, 257, 255), (F32, 1, 256, 3, 255), (F32, 4, 16, 65, 300),
]


def _rope(x, pos):
    half = x.shape[-1] // 2
    ang = pos[:, None, None] * THETA ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _norm(x):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v).replace("torch.", "") for v in c))
def test_step_against_64_bits(case):
    L = need_gpu()
    dt, H, dh, B, keys = case
    d, ff = H * dh, 64 * max(1, H * dh // 64)
    log(f"[decode attention] {case}")
    g = torch.Generator(device="cuda").manual_seed(5)

    def rnd(*shape, std):
        return (torch.randn(*shape, device="cuda", generator=g) * std).to(dt)

    w = {k: rnd(d, d, std=d ** -0.5) for k in ("wq", "wk", "wv", "wo")}
    w.update(wg=rnd(ff, d, std=0.02), wu=rnd(ff, d, std=0.02), wd=rnd(d, ff, std=0.02))
    w.update({k: torch.ones(d, device="cuda") for k in ("attn_norm", "ffn_norm")})
    cfg = L.decoder_cfg(1, d, H, ff, L.BF16 if dt == BF else L.F32, EPS, THETA)
    lens = np.array([keys - b % 3 if b % 5 else keys for b in range(B)], np.int32)
    kv = L.kv_cache(cfg, B, keys + 1, "cuda")
    kv["k"].copy_(rnd(*kv["k"].shape, std=4.0))  # sharp: a few keys carry the result
    kv["v"].copy_(rnd(*kv["v"].shape, std=2.0))
    x = rnd(B, d, std=0.3)
    K, V = (kv[t][0].double().view(B, keys + 1, H, dh) for t in ("k", "v"))
    h = L.decode_step(cfg, [w], lens, x, kv)[0]
    f = {k: t.double() for k, t in w.items()}
    pos = torch.from_numpy(lens).cuda().long()
    xd = x.double()
    xn = _norm(xd)
    q, k = (_rope((xn @ f[t].T).view(B, H, dh), pos.double()) for t in ("wq", "wk"))
    at = torch.arange(B, device="cuda")
    K[at, pos], V[at, pos] = k, (xn @ f["wv"].T).view(B, H, dh)
    z = torch.matmul(K.transpose(1, 2), q[..., None])[..., 0] / math.sqrt(dh)
    z = z.masked_fill(torch.arange(keys + 1, device="cuda")[None, None] > pos[:, None, None], -math.inf)
    o = torch.matmul(torch.softmax(z, -1)[:, :, None], V.transpose(1, 2))[:, :, 0].reshape(B, d)
    y = xd + o @ f["wo"].T
    yn = _norm(y)
    ref = y + (torch.nn.functional.silu(yn @ f["wg"].T) * (yn @ f["wu"].T)) @ f["wd"].T
    assert float((ref - xd).abs().max()) > 0.5  # the attention is most of the result
    e = float((h.double() - ref).abs().max() / ref.abs().max())
    log(f"  {e:.2e}")
    assert e <= (2e-2 if dt == BF else 1e-4)

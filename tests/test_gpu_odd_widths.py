"""Widths that are odd multiples of 64 at more than 256 rows (the LDS-staged GEMM with 64 columns
per block): the vocabulary of a decode step and of the online controller's lens, and the
projector's widths.  fp32 sums of bf16 products against 64 bits of the same inputs."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import get_workload
from gpu_common import need_gpu, log
from test_gpu_prefill import _oracle_weights, _x


def _setup(L, rows, n_layers=2):
    dec = dataclasses.replace(get_workload("llava15_7b").dec, L=n_layers, d=256, H=2, d_ff=320)
    W = [{k: torch.from_numpy(v).to("cuda", torch.float32 if "norm" in k else torch.bfloat16)
          for k, v in _oracle_weights(dec, n_layers)(l).items()} for l in range(n_layers)]
    return dec, W, L.decoder_cfg(n_layers, dec.d, dec.H, dec.d_ff, L.BF16, dec.eps, dec.theta), _x(dec, rows, 3)


def _rows(shape, seed, std):
    return (torch.randn(*shape, generator=torch.Generator().manual_seed(seed)) * std).bfloat16()


@pytest.mark.gpu
def test_decode_head_of_260_samples():
    L = need_gpu()
    B, V = 260, 192
    log(f"[odd widths] head, {B} samples, V={V}")
    dec, W, cfg, x = _setup(L, B)
    kv = L.kv_cache(cfg, B, 4, "cuda")
    wu, fn = _rows((V, dec.d), 5, 0.05), 1 + 0.1 * _rows((dec.d,), 6, 1.0).float()
    h, logits, nxt = L.decode_step(cfg, W, np.zeros(B, np.int32), x.cuda(), kv, fn.cuda(), wu.cuda())
    hd = h.cpu().double()
    xn = (hd / torch.sqrt((hd * hd).mean(1, keepdim=True) + dec.eps) * fn.double()).bfloat16().double()
    ref = xn @ wu.double().T
    # a norm that rounds to the other bf16 moves a logit by one rounding (2^-8) of one of 256 products
    assert float((logits.cpu() - ref).abs().max() / ref.abs().max()) <= 2e-3
    assert torch.equal(nxt.cpu().long(), logits.cpu().argmax(1))


@pytest.mark.gpu
def test_online_lens_of_400_rows():
    L = need_gpu()
    rows, n_text, V = 400, 32, 320
    log(f"[odd widths] lens, {rows} rows, V={V}")
    dec, W, cfg, x = _setup(L, rows)
    wu = _rows((V, dec.d), 5, 0.2)
    # the visual rows point away from the text rows and their lens is sharp, so that no score is clamped to 0
    u = _rows((1, dec.d), 12, 1.0).float()
    x = torch.cat([x[:rows - n_text].float() - 1.5 * u, x[rows - n_text:].float() + u]).bfloat16()
    sel, target = L.slc_policy(np.array([0.1, 0.1], np.float32), np.array([10.0, 10.0], np.float32))
    _, _, admit, s_sa = L.prefill_online(cfg, W, np.array([0, rows], np.int32), x.cuda(), n_text, wu.cuda(), sel, target,
                                         3.0, 1.0, 1e6)
    assert (admit[:] == -1).all()
    h = x.double()
    logp = torch.log_softmax(h @ wu.double().T, 1)
    ent = -(logp.exp() * logp).sum(1) / np.log(V)
    text = h[rows - n_text:].mean(0)
    cos = (h @ text) / (h.norm(dim=1) * text.norm())
    ref = (1 - ent - (1 + cos) / 2).clamp_min(0)[:rows - n_text]
    assert float(ref.min()) > 0.01
    assert float((s_sa[0, :rows - n_text].cpu() - ref).abs().max()) <= 1e-4


@pytest.mark.gpu
def test_projector_of_260_rows():
    L = need_gpu()
    n, keep, din, dh, do = 576, 256, 192, 64, 320
    log(f"[odd widths] projector {din}-{dh}-{do}")
    g = torch.Generator().manual_seed(3)
    rank = torch.rand(1, n, generator=g).argsort(1).argsort(1)
    cluster = torch.where(rank < 128, -1, torch.randint(0, 4, (1, n), generator=g)).int()
    score = torch.rand(1, n, generator=g)
    ft, text = _rows((1, n + 1, din), 4, 1.0), _rows((1, 8, do), 7, 1.0)
    p = {"w1": _rows((dh, din), 8, 0.1), "b1": _rows((dh,), 9, 0.1).float(), "w2": _rows((do, dh), 10, 0.1),
         "b2": _rows((do,), 11, 0.1).float()}
    sel = L.select(cluster.cuda(), score.cuda(), 128, keep - 128, quota_mode=1, text=text.cuda(), text_only=True)
    L.project_kept(sel, ft.cuda(), {k: v.cuda() for k, v in p.items()}, 1, 8)
    idx = sel["idx"][0, :int(sel["count"][0])].cpu().long()
    assert len(idx) == keep
    hid = ft[0, 1:][idx].double() @ p["w1"].double().T + p["b1"].double()
    ref = (torch.nn.functional.gelu(hid).bfloat16().double() @ p["w2"].double().T) + p["b2"].double()
    got = sel["x"][:keep].cpu().double()
    # the output is rounded to bf16 (2^-9 of a value) and a hidden value may round to the other bf16
    assert float((got - ref).abs().max() / ref.abs().max()) <= 1e-2

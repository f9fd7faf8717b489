"""Scoring and selection at the edges of their kernels' tiles: row counts around a wave, a
64-index register of the top-k, a staged chunk of rows and a 32-row tile; widths that are not
a multiple of 64; one and three tapped layers; cluster counts 1 to 8.  Bars as in
test_gpu_score.py (anchors, clusters and kept indices exact, s and m within 1e-5)."""
import numpy as np
import pytest
import torch

from synth.configs import ScoreCfg
from synth.vision import llava_taps
from gpu_common import need_gpu, oracle_tiles, log

SHAPES = [
    # G, n, d_v, taps, keep, K, dtype
    (1, 33, 8, 1, 20, 3, "bf16"),
    (2, 64, 72, 2, 40, 4, "bf16"),
    (1, 65, 136, 3, 10, 1, "f32"),
    (3, 100, 64, 2, 100, 8, "bf16"),
    (1, 577, 1160, 1, 300, 2, "bf16"),
    (1, 1024, 520, 2, 900, 5, "f32"),
    (1, 1025, 256, 2, 64, 4, "bf16"),
    (1, 2100, 384, 2, 700, 4, "bf16"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_score_and_select_edges(shape):
    L = need_gpu()
    G, n, d, taps, keep, K, dt = shape
    log(f"[score paths] {shape}")
    cfg = ScoreCfg(G=G, n=n, H=3, d_v=d, layers=tuple(range(12, 12 + taps)), feat_dtype="bf16", keep=keep, K=K)
    attn, feats = llava_taps(cfg, 5)
    if dt == "f32":
        feats = [f.float() for f in feats]
    na, nc = L.budget(keep)
    out = L.score(attn.cuda(), [f.cuda() for f in feats], na, K, 10)
    ref = oracle_tiles(attn, feats, keep, K=K)
    for g, o in enumerate(ref):
        assert o["margin"].size == 0 or o["margin"].min() > 1e-5, "input too close to a K-means tie"
        assert np.array_equal(out["a"][g].cpu().numpy(), o["a"])
        assert np.array_equal(out["cluster"][g].cpu().numpy(), o["cluster"])
        s, m, rest = out["s"][g].cpu().numpy(), out["m"][g].cpu().numpy(), o["cluster"] >= 0
        assert np.all(np.isinf(s[~rest]))
        assert np.max(np.abs(s[rest] - o["s"][rest]) / np.maximum(1, np.abs(o["s"][rest])), initial=0) <= 1e-5
        assert np.max(np.abs(m - o["mvec"])) <= 1e-5
    from oracle import msv_prune as mp
    for mode, name in ((0, "literal"), (1, "exact")):
        sel = L.select(out["cluster"], out["s"], na, nc, K, mode)
        for g in range(G):
            idx, _ = mp.select(out["cluster"][g].cpu().numpy(), out["s"][g].cpu().numpy(), nc, K, name)
            assert sel["idx"][g, :int(sel["count"][g])].tolist() == idx
            assert bool((sel["idx"][g, int(sel["count"][g]):] == -1).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 64, 130, 1024, 3000])
def test_select_special_scores(n):
    """Equal scores, infinities, NaN, signed zeros: the order of the float keys, then the index."""
    L = need_gpu()
    log(f"[select] special scores n={n}")
    r = np.random.default_rng(n)
    s = r.choice(np.array([0.0, -0.0, 1.0, -1.0, np.inf, -np.inf, np.nan, 1e-40], np.float32), n)
    cl = r.integers(-1, 4, n).astype(np.int32)
    n_cmp = n // 2
    sel = L.select(torch.from_numpy(cl)[None].cuda(), torch.from_numpy(s)[None].cuda(), int((cl < 0).sum()), n_cmp, 4, 1)
    bits = np.where(s == 0, np.float32(0), s).view(np.uint32).astype(np.int64)
    key = np.where(bits >> 31, 0xFFFFFFFF - bits, bits | 0x80000000)
    from oracle import msv_prune as mp
    quota = mp.quotas([int((cl == k).sum()) for k in range(4)], n_cmp, "exact")
    want = set(np.nonzero(cl < 0)[0].tolist())
    for k in range(4):
        i = np.nonzero(cl == k)[0]
        want |= set(i[np.argsort(key[i], kind="stable")][:quota[k]].tolist())
    assert sel["idx"][0, :int(sel["count"][0])].tolist() == sorted(want)


@pytest.mark.gpu
@pytest.mark.parametrize("G,K", [(60, 4), (100, 8)])
def test_tiles_of_a_large_batch_have_their_own_bits(G, K):
    """1080 and 1800 similarity blocks, two to a CU: every tile's scores are those of the tile alone,
    pass after pass (an LDS stage refilled while a wave still reads it shows here first)."""
    L = need_gpu()
    log(f"[score paths] {G} tiles of 4, K={K}")
    cfg = ScoreCfg(G=4, n=576, H=3, d_v=1024, layers=(12, 24), feat_dtype="bf16", keep=128, K=K)
    attn, feats = llava_taps(cfg, 9)
    attn, feats = attn.cuda(), [f.cuda() for f in feats]
    alone = [L.score(attn[g:g + 1], [f[g:g + 1] for f in feats], 89, K, 10) for g in range(4)]
    of = [g % 4 for g in range(G)]
    many = attn[of].contiguous(), [f[of].contiguous() for f in feats]
    for _ in range(10):
        out = L.score(*many, 89, K, 10)
        for key in ("a", "cluster", "s", "m"):
            want = torch.cat([alone[g][key] for g in of])
            assert torch.equal(out[key], want), key

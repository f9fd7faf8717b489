"""Pipeline.step on the host (no GPU): with exact quotas the step plans and launches the prefill
while the device still reads its inputs, so it must wait for that reading however it is left."""
import numpy as np
import pytest
import torch

from paper_2609_34977_amd import _lib, pipeline
from paper_2609_34977_amd.pipeline import Pipeline, SkipPolicy


class _Event:
    def __init__(self, log):
        self.log = log

    def record(self, stream):
        self.log.append("record")

    def synchronize(self):
        self.log.append("wait")


def _pipeline(log, monkeypatch, prefill):
    p = Pipeline.__new__(Pipeline)
    p.G, p.n, p.K, p.B, p.tps = 1, 8, 2, 1, 1
    p.n_anchor, p.n_cmp, p.cap, p.kmeans_iter, p.n_text, p.quota_mode = 3, 2, 5, 1, 4, 1
    p.dec, p.device, p.projector, p.online_ws = _lib.decoder_cfg(1, 4, 1, 4, _lib.F32, 1e-5, 1e4), "cpu", None, None
    p.h, p.prefill_ws, p.wtable, p.max_rows = torch.zeros(9, 4), None, None, 9
    p.inputs_read = _Event(log)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: None)
    monkeypatch.setattr(pipeline._lib, "score", lambda *a: {"cluster": None, "s": None})
    monkeypatch.setattr(pipeline._lib, "select", lambda *a, **k: {"x": torch.zeros(9, 4)})
    monkeypatch.setattr(pipeline._lib, "prefill", prefill)
    return p


MASK = SkipPolicy("layer_mask", layer_mask=np.zeros((1, 2), bool))


def test_waits_for_the_inputs(monkeypatch):
    log = []
    p = _pipeline(log, monkeypatch, lambda *a, **k: log.append("prefill") or "h")
    r = p.step(None, None, None, None, MASK)
    assert log == ["record", "prefill", "wait"]
    assert r["h"] == "h" and r["cu"].tolist() == [0, 9] and r["codes"].shape == (1, 9)


@pytest.mark.parametrize("where", ["plan", "prefill"])
def test_waits_for_the_inputs_when_the_step_fails(monkeypatch, where):
    def prefill(*a, **k):
        raise RuntimeError("prefill")

    log = []
    p = _pipeline(log, monkeypatch, prefill)
    with pytest.raises(ValueError if where == "plan" else RuntimeError):
        p.step(None, None, None, None, SkipPolicy("unknown") if where == "plan" else MASK)
    assert log == ["record", "wait"]

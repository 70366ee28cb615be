"""The prompt tests on the GPU can fail: mistakes planted in the oracle move the
readouts of their models by several times what they allow."""
import numpy as np

from oracle import model as OM
from prompt_models import REL, SINK_NATS, readouts, rel, sink_model, sink_prompt, sink_spec


def test_small_weights_show(monkeypatch):
    """Weights rounded to fp16 against the largest of the whole row: what lies 2^-25 below it is gone."""
    spec = sink_spec()
    w = sink_model(spec)
    pr = sink_prompt(spec)
    want = readouts(OM.LoopedLM(spec, w), pr, 5)

    def rounded(q, K, V, qp, kp):
        s = np.einsum("qhd,khd->hqk", q, K) / np.sqrt(q.shape[-1])
        s = np.where(np.asarray(kp)[None, None] > np.asarray(qp)[None, :, None], -np.inf, s)
        p = np.exp(s - s.max(-1, keepdims=True)).astype(np.float16).astype(np.float64)
        return np.einsum("hqk,khd->qhd", p / p.sum(-1, keepdims=True), V)

    with monkeypatch.context() as m:
        m.setattr(OM, "causal_attention", rounded)
        bad = OM.LoopedLM(spec, w)
        node = bad.prefill(pr)
    assert rel(readouts(bad, pr, 5, node), want).max() > 5 * (REL + 2 * SINK_NATS * 2.0 ** -11)

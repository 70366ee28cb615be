"""The prompt tests on the GPU can fail: mistakes planted in the oracle move the
readouts of their models by several times what they allow."""
import numpy as np

from oracle import model as OM
from prompt_models import REL, SINK_NATS, near_model, near_spec, readouts, rel, sink_model, sink_prompt, sink_spec

FIRST = 2048                                                    # positions of the first prompt pass


def second_pass(f):
    """causal_attention with f(q, K, V, qpos, kpos) for the queries of the second pass."""
    whole = OM.causal_attention

    def g(q, K, V, qp, kp):
        a, i = whole(q, K, V, qp, kp), np.asarray(qp) >= FIRST
        if len(qp) > 1 and i.any():
            a[i] = f(whole, q[i], K, V, np.asarray(qp)[i], np.asarray(kp))
        return a
    return g


MISTAKES = {
    "mask one late": lambda att, q, K, V, qp, kp: att(q, K, V, qp + 1, kp),
    "mask one early": lambda att, q, K, V, qp, kp: att(q, K, V, qp - 1, kp),
    "blind to the first pass": lambda att, q, K, V, qp, kp: att(q, K[FIRST:], V[FIRST:], qp, kp[FIRST:]),
    "a tile of the first pass missing": lambda att, q, K, V, qp, kp: att(
        q, np.delete(K, np.s_[FIRST - 64:FIRST], 0), np.delete(V, np.s_[FIRST - 64:FIRST], 0), qp,
        np.delete(kp, np.s_[FIRST - 64:FIRST])),
}


def test_second_pass_mistakes_show(monkeypatch):
    n = 2060
    spec = near_spec()
    w = near_model(spec)
    pr = [int(t) for t in np.random.default_rng(n).integers(0, spec.vocab, n)]
    lm = OM.LoopedLM(spec, w)
    want = readouts(lm, pr, 5)
    for name, f in MISTAKES.items():
        with monkeypatch.context() as m:
            m.setattr(OM, "causal_attention", second_pass(f))
            bad = OM.LoopedLM(spec, w)
            node = bad.prefill(pr)
        assert rel(readouts(bad, pr, 5, node), want).max() > 5 * REL, name
    # positions of the second pass rotated, or stored, as those of the first
    rope = OM.rope
    with monkeypatch.context() as m:
        m.setattr(OM, "rope", lambda x, pos, base: rope(x, np.where(np.asarray(pos) >= FIRST, np.asarray(pos) - FIRST, pos), base))
        bad = OM.LoopedLM(spec, w)
        node = bad.prefill(pr)
    assert rel(readouts(bad, pr, 5, node), want).max() > 5 * REL
    for lo, hi in ((FIRST, n), (FIRST - 64, FIRST)):
        bad = OM.LoopedLM(spec, w)
        node = bad.prefill(pr)
        for k, v in node.kv.values():
            k[lo:hi] = v[lo:hi] = 0.0
        assert rel(readouts(bad, pr, 5, node), want).max() > 5 * REL


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

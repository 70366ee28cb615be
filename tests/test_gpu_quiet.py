"""Decode loops that replay a shorter step between two readouts (models with
prelude or coda blocks) against the same handle stepped with the whole step."""
import numpy as np
import pytest

from gpu_common import log, model, prompt

pytestmark = pytest.mark.gpu

COUNTS = ("steps", "n_acc1", "n_acc2", "n_restart", "gate_eval", "gate_open", "spawn_refused")


@pytest.mark.parametrize("R,d1,d2,temperature,Q,second", [
    (8, 4, 0, 0.0, 1, None), (16, 4, 8, 0.0, 1, (8, 0)), (16, 8, 12, 0.0, 1, (12, 0)), (15, 5, 10, 0.0, 1, None),
    (16, 8, 12, 1.0, 1, None), (12, 6, 0, 0.8, 1, None),
    # whole steps, throughout or up to the switch
    (16, 8, 12, 0.0, 3, None), (8, 4, 6, 0.0, 1, (4, 0)), (16, 6, 8, 0.0, 1, (8, 0))])
def test_decode_equals_single_steps(R, d1, d2, temperature, Q, second):
    """Integer outcomes of two routes over the same kernels: equal.  One
    sequence whose depths share a divisor of at least 4 takes the short steps
    (from the smallest such divisor up), others the whole ones; a switch of the
    depths moves the next readout, and the route, between two calls."""
    check(*model("small_raven", R=R), R, d1, d2, temperature, Q, second)


@pytest.mark.parametrize("R,d1", [(8, 4), (10, 5), (12, 6)])
def test_decode_of_a_model_without_coda_equals_single_steps(R, d1):
    """Its short steps save fewer launches: from a gap of 5 up."""
    check(*model("small_raven", R=R, n_coda=0), R, d1, 0, 0.0, 1, None)


def check(spec, w, R, d1, d2, temperature, Q, second):
    from paper_2609_17184_amd import Decoder
    kw = {"temperature": temperature, "top_p": 0.9, "seed": 5} if temperature else {}
    N = 21
    log(f"[quiet] R={R} d1={d1} d2={d2} T={temperature} Q={Q} second={second}")

    def start():
        dec = Decoder(spec, w, R=spec.R, d1=d1, d2=d2, max_seqs=Q, max_ctx=128, max_slots=64, **kw)
        for q in range(Q):
            dec.prefill(q, prompt(spec, 11 + 5 * q, seq=q))
        return dec

    dec = start()
    got = [list(t) for t in dec.decode(N)]
    stats = dec.stats()
    if second:
        dec.set_depths(*second)
        for q, t in enumerate(dec.decode(N)):
            got[q] += list(t)
    for q in range(Q):
        dec.rewind(q)
    vanilla = [list(t) for t in dec.vanilla_decode(len(got[0]))] if not temperature else None
    dec.close()

    ref = start()
    toks = [[] for _ in range(Q)]
    for _ in range(spec.R * (N + 2)):
        t, _ = ref.decode_step()
        for q in range(Q):
            if t[q] >= 0 and len(toks[q]) < N:
                toks[q].append(int(t[q]))
        if all(len(t) == N for t in toks):
            break
    assert [g[:N] for g in got] == toks
    if Q == 1:
        st = ref.stats()
        assert {k: stats[k] for k in COUNTS} == {k: st[k] for k in COUNTS}
    ref.close()
    if vanilla:
        assert got == vanilla

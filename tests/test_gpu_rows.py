"""GPU: the weight stream of handles with more than 16 branch slots (17 to 64
rows), against the fp64 oracle and across row counts."""
import numpy as np
import pytest

import synth
from gpu_common import TOL, log, model, oracle_lm, prompt
from oracle import model as OM
from paper_2609_17184_amd import Decoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [20, 64])
def test_deep_loads_match_oracle(slots):
    """K = 5120 and 320 / 480 workgroups: the launches that load further ahead (QKV with two feature tiles per
    workgroup, O with one), for 32- and 64-row instantiations; the FFN and the head take the others."""
    spec = synth.ModelSpec(5120, 40, 128, 96, 304, 0, 1, 0, R=2, alpha=0.3)
    w = synth.make_weights(spec, seed=0)
    lm = OM.LoopedLM(spec, w)
    pr = [int(t) for t in prompt(spec, 19)]
    node = lm.prefill(pr)
    tok = int(np.argmax(lm.logits(node, spec.R)))
    dec = Decoder(spec, w, R=2, d1=1, d2=0, max_seqs=1, max_ctx=64, max_slots=slots)
    dec.prefill(0, pr)
    log(f"[rows] {slots} slots")
    lg, _ = dec.forced_readout(0, [tok])
    node = lm.extend(node, tok)
    for r in (1, 2):
        err = float(np.abs(lg[0, r - 1] - lm.logits(node, r)).max())
        assert err < TOL["bf16"], (slots, r, err)
    dec.close()


@pytest.mark.parametrize("name,seqs", [("small_bf16", 17), ("small_bf16", 33), ("small_raven", 50), ("tiny", 64)])
def test_rows_do_not_depend_on_each_other(name, seqs):
    """Vanilla decoding of `seqs` sequences in one pass (two to four row tiles, the last one ragged) commits the tokens
    that each sequence gets alone in a handle of the same slots, and a few of them match the oracle's readout."""
    spec, w = model(name)
    kw = dict(R=spec.R, d1=spec.R - 1, d2=0, max_ctx=40, max_slots=64)
    dec = Decoder(spec, w, max_seqs=seqs, **kw)
    prompts = [prompt(spec, 3 + q % 7, seq=q) for q in range(seqs)]
    for q, pr in enumerate(prompts):
        dec.prefill(q, pr)
    got = dec.vanilla_decode(3)
    dec.close()
    one = Decoder(spec, w, max_seqs=1, **kw)
    for q in (0, 15, 16, seqs - 1):
        log(f"[rows] {name} {seqs} sequences: sequence {q} alone")
        one.prefill(0, prompts[q])
        assert np.array_equal(one.vanilla_decode(3)[0], got[q]), q
    one.close()

"""GPU: prompt passes at the edges of their tiles, against the fp64 oracle.

The readouts after a prompt depend on every key and value that its pass wrote,
at every depth: one teacher-forced position behind the prompt is compared at
all depths, and the prompt's own first token.  Tolerances are the logits'
(gpu_common.TOL: fp16 operands with fp32 sums, or fp32 throughout)."""
import numpy as np
import pytest

import synth
from gpu_common import MARGIN, TOL, log, model, oracle_lm, prompt
from oracle import model as OM
from paper_2609_17184_amd import Decoder
from prompt_models import REL, SINK_NATS, near_model, near_spec, readouts, readouts64, rel, sink_model, sink_prompt, sink_spec

pytestmark = pytest.mark.gpu


def check(spec, w, lm, n, max_ctx):
    pr = [int(t) for t in prompt(spec, n)]
    log(f"[prefill] {spec.hidden} wide {spec.weight_dtype}, {n} positions")
    node = lm.prefill(pr)
    z0 = lm.logits(node, spec.R)
    d2 = 2 if spec.R > 2 else 0
    dec = Decoder(spec, w, R=spec.R, d1=1, d2=d2, max_seqs=1, max_ctx=max_ctx)
    tok = int(np.argmax(z0))
    first = dec.prefill(0, pr)
    top = np.sort(z0)[-2:]
    if top[1] - top[0] > MARGIN[spec.weight_dtype]:
        assert first == tok
    lg, _ = dec.forced_readout(0, [tok])
    node = lm.extend(node, tok)
    for r in range(1, spec.R + 1):
        err = float(np.abs(lg[0, r - 1] - lm.logits(node, r)).max())
        assert err < TOL[spec.weight_dtype], (n, r, err)
    dec.close()


@pytest.mark.parametrize("name", ["tiny", "small_bf16", "small_raven"])
@pytest.mark.parametrize("n", [1, 2, 16, 17, 63, 64, 65, 129])
def test_prompt_lengths(name, n):
    """Row tiles of 16 and blocks of 64, one row short, full and one over; keys of 64 positions."""
    spec, w = model(name)
    check(spec, w, oracle_lm(name), n, 160)


@pytest.mark.parametrize("n", [2048, 2049, 2111])
def test_prompt_of_several_passes(n):
    """A pass holds 2048 positions, the next one goes on behind them, in prelude and coda blocks too.  (Each key weighs
    little in this model; test_prompt_near_keys sees what the second pass does.)"""
    spec, w = model("small_raven", R=2)
    check(spec, w, oracle_lm("small_raven", R=2), n, 2200)


def test_prompt_tiles_of_128():
    """Every GEMM of a block over 2000 rows at this width has 256 tiles of 128 x 128 or more (the rule's line is 200),
    the last row block ragged."""
    spec = synth.ModelSpec(2048, 16, 128, 1024, 512, 0, 1, 0, R=2, alpha=0.3)
    w = synth.make_weights(spec, seed=0)
    check(spec, w, OM.LoopedLM(spec, w), 2000, 2048)


@pytest.mark.parametrize("dh", [16, 32, 64])
@pytest.mark.parametrize("n", [15, 64, 130])
def test_prompt_head_sizes(dh, n):
    """The causal attention of a 16-bit prompt for the head sizes the presets do not have (96 and 128 are above)."""
    spec = synth.ModelSpec(128, 128 // dh, dh, 256, 304, 0, 2, 0, R=3, alpha=0.3)
    w = synth.make_weights(spec, seed=0)
    check(spec, w, OM.LoopedLM(spec, w), n, 160)


def test_prompt_of_many_query_blocks():
    """2100 positions of 16 heads, keys of 33 tiles, two passes.  (As above: single keys weigh little here.)"""
    spec = synth.ModelSpec(256, 16, 16, 256, 304, 0, 1, 0, R=2, alpha=0.3)
    w = synth.make_weights(spec, seed=0)
    check(spec, w, OM.LoopedLM(spec, w), 2100, 2200)


def off(spec, w, pr, tok, max_ctx):
    """Relative error of the readouts of one position behind a prompt."""
    want = readouts64(spec, w, pr + [tok]) if len(pr) > 2200 else readouts(OM.LoopedLM(spec, w), pr, tok)
    dec = Decoder(spec, w, R=spec.R, d1=1, d2=0, max_seqs=1, max_ctx=max_ctx)
    dec.prefill(0, pr)
    got, _ = dec.forced_readout(0, [tok])
    dec.close()
    e = rel(got[0], want)
    log(f"[prefill] {len(pr)} positions of {spec.n_heads} x {spec.head_dim}: off by {e}")
    return e.max()


@pytest.mark.parametrize("dh", [16, 64, 96, 128])
def test_prompt_small_weights(dh):
    """Attention outputs made of weights 2^-27 below the row's largest: a key of no value far above the others.  A
    score of SINK_NATS is a sum of products of two factors rounded at 2^-11 each."""
    spec = sink_spec(dh=dh)
    assert off(spec, sink_model(spec), sink_prompt(spec), 5, 200) < REL + 2 * SINK_NATS * 2.0 ** -11


@pytest.mark.parametrize("H,dh,n", [(1, 96, 2049), (1, 96, 2060), (1, 96, 2111), (16, 16, 2111)])
def test_prompt_near_keys(H, dh, n):
    """Readouts that hang on the keys just before them, so on every position of a second pass and on its view of the
    first."""
    spec = near_spec(H, dh)
    pr = [int(t) for t in np.random.default_rng(n).integers(0, spec.vocab, n)]
    assert off(spec, near_model(spec), pr, 5, n + 32) < REL


@pytest.mark.parametrize("H,dh,n", [(64, 16, 5567), (64, 16, 5632), (64, 16, 6130), (64, 32, 6144), (64, 64, 6050),
                                    (48, 96, 6144), (48, 128, 6100)])
def test_prompt_query_blocks_of_128(H, dh, n):
    """32 queries per wave: behind 4096 positions from 768 blocks of 128 queries on (64 heads: 1409 rows), the last one
    half empty, ragged or full."""
    spec = near_spec(H, dh, F=256, V=304)
    w = near_model(spec)
    pr = [int(t) for t in np.random.default_rng(n).integers(0, spec.vocab, n)]
    assert off(spec, w, pr, 5, n + 32) < REL


def test_float64_reference_equals_the_oracle():
    spec = near_spec(2, 32, F=256, V=304)
    w = near_model(spec)
    pr = [int(t) for t in np.random.default_rng(0).integers(0, spec.vocab, 90)]
    assert rel(readouts64(spec, w, pr + [5]), readouts(OM.LoopedLM(spec, w), pr, 5)).max() < 1e-12

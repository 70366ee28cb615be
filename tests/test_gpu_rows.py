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
    """One live row at K = 5120 in the 32- and 64-row instantiations: QKV with two feature tiles per workgroup, the
    others with one."""
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
    that each sequence gets alone in a handle of the same slots."""
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


def step_and_read(dec, prompts, depth, seqs):
    """Prefills every sequence, advances all of them `depth` steps in passes of that many rows and returns the readouts
    of the given sequences' roots at that depth: of the states that the passes left."""
    first = [dec.prefill(q, pr) for q, pr in enumerate(prompts)]
    for _ in range(depth):
        dec.decode_step()
    out = {}
    for slot, info, _ in dec.branches():
        if info["parent"] == -1 and info["seq"] in seqs:
            assert info["depth"] == depth
            out[info["seq"]] = dec.debug_readout(slot, depth)
    return first, out


@pytest.mark.parametrize("name,seqs,slots", [
    ("wide", 20, 32), ("wide", 50, 64), ("wide", 64, 64), ("wide_f32", 40, 64), ("ragged_f32", 33, 64),
    ("small_bf16", 33, 64), ("small_raven", 50, 64), ("tiny", 64, 64)])
def test_wide_passes_match_oracle(name, seqs, slots):
    """Readouts of sequences from every row tile after two passes of `seqs` live rows: within tolerance of the oracle,
    and bit for bit those of the sequence alone in a handle of the same slots.  wide: QKV with two feature tiles and
    gate/up six k steps ahead (128 of them); wide_f32: the same at its fp32 threshold of 160 steps; ragged_f32: the last
    of 30 tiles ends a workgroup, 15 k steps in shares of 3 and 4."""
    spec = {"wide": synth.ModelSpec(4096, 32, 128, 512, 304, 0, 1, 0, R=3, alpha=0.3),
            "wide_f32": synth.ModelSpec(2560, 40, 64, 256, 304, 0, 1, 0, R=3, weight_dtype="f32", alpha=0.3),
            "ragged_f32": synth.ModelSpec(480, 30, 16, 224, 301, 0, 1, 0, R=3, weight_dtype="f32", alpha=0.3),
            "small_bf16": synth.preset("small_bf16", R=3), "small_raven": synth.preset("small_raven", R=3),
            "tiny": synth.preset("tiny", R=3)}[name]
    w = synth.make_weights(spec, seed=0)
    kw = dict(R=3, d1=2, d2=0, max_ctx=40, max_slots=slots)
    prompts = [prompt(spec, 3 + q % 7, seq=q) for q in range(seqs)]
    look = sorted({0, 15, 16, 31, 32, 47, 48, seqs - 1} & set(range(seqs)))
    dec = Decoder(spec, w, max_seqs=seqs, **kw)
    log(f"[rows] {name}: {seqs} live rows")
    first, got = step_and_read(dec, prompts, 2, look)
    dec.close()
    one = Decoder(spec, w, max_seqs=1, **kw)
    lm = OM.LoopedLM(spec, w)
    for q in look:
        _, alone = step_and_read(one, prompts[q:q + 1], 2, {0})
        assert np.array_equal(alone[0], got[q]), q
        want = lm.logits(lm.extend(lm.prefill([int(t) for t in prompts[q]]), first[q]), 2)
        err = float(np.abs(got[q] - want).max())
        assert err < TOL[spec.weight_dtype], (q, err)
    one.close()


@pytest.mark.parametrize("seqs", [20, 50])
def test_wide_head_matches_oracle(seqs):
    """The head with two feature tiles per workgroup (775 tiles, the last one ragged) over every live row: the tokens
    of a vanilla step, where the oracle's two largest logits lie apart."""
    spec = synth.ModelSpec(256, 2, 128, 256, 12390, 0, 1, 0, R=2, alpha=0.3)
    w = synth.make_weights(spec, seed=0)
    dec = Decoder(spec, w, R=2, d1=1, d2=0, max_seqs=seqs, max_ctx=40, max_slots=64 if seqs > 32 else 32)
    prompts = [prompt(spec, 3 + q % 7, seq=q) for q in range(seqs)]
    first = [dec.prefill(q, pr) for q, pr in enumerate(prompts)]
    toks = dec.vanilla_decode(1)
    dec.close()
    lm, seen = OM.LoopedLM(spec, w), 0
    log(f"[rows] head: {seqs} live rows")
    for q in range(seqs):
        z = lm.logits(lm.extend(lm.prefill([int(t) for t in prompts[q]]), first[q]), 2)
        top = np.sort(z)[-2:]
        if top[1] - top[0] > 2 * 8 * 2.0 ** -11 * top[1]:        # eight roundings to fp16 on either side
            assert toks[q][0] == int(np.argmax(z)), q
            seen += 1
    assert seen >= seqs // 2

"""Performance cases of the LoopSpec library: the work its users have it do, through its public entry points.

Four kinds of call, on looped models of this repository's shapes:

  cascade   the standalone proposal / verification decisions of given readout logits
  prefill   a prompt into the caches of every depth, then its readout at every depth (what a serving loop or the depth
            planner does with a new prompt)
  readout   teacher-forced readouts of a continuation at every depth (the vanilla schedule, one position at a time)
  decode    LoopSpec decoding of prefilled sequences, greedy or sampled, plus the readout of each root's newest token

The models are random with the one property of trained ones that decides what a decode does: confident, agreeing
readouts.  Embeddings have unit entries, the blocks' residual branches are scaled so that their sum over all depths
about equals the embedding (alpha), attention scores have a standard deviation of about 2, and the LM head's row for a
token's successor points along the token's embedding with about 0.99 of the probability.  So greedy and sampled
continuations do not hang on the last bit of a logit, while half of every logit's variance comes from the blocks.
"""
import functools
import math
import types

import numpy as np
import torch

from paper_2609_17184_amd import Decoder, worst_case_branches
from paper_2609_17184_amd.binding import cascade as run_cascade

DEV = "cuda:0"

# widths of the model families: the tiny fp32 decoder, the Ouro and Raven shapes, and a small ragged one (96-wide heads)
WIDTHS = {
    "tiny": dict(hidden=256, n_heads=4, head_dim=64, ffn=1024, vocab=4096, weight_dtype="f32", tied_head=True),
    "ragged": dict(hidden=192, n_heads=2, head_dim=96, ffn=512, vocab=800, weight_dtype="bf16", tied_head=False),
    "ouro": dict(hidden=2048, n_heads=16, head_dim=128, ffn=5632, vocab=49152, weight_dtype="bf16", tied_head=False),
    "raven": dict(hidden=5280, n_heads=55, head_dim=96, ffn=17920, vocab=65536, weight_dtype="bf16", tied_head=False),
}


def model_case(name, kind, width, blocks, R, d1, d2, seqs, prompt, tokens, temperature=0.0, top_p=1.0, per_kernel=False,
               shared_prefix=False):
    """`blocks`: prelude/core/coda block counts; `prompt`: tokens of the longest prompt; `tokens`: generated or forced."""
    return dict(name=name, kind=kind, width=width, blocks=blocks, R=R, d1=d1, d2=d2, seqs=seqs, prompt=prompt,
                tokens=tokens, temperature=temperature, top_p=top_p, per_kernel=per_kernel, shared_prefix=shared_prefix)


def listed():
    return [
        # the smallest call: four positions' decisions over a small vocabulary, in a loop that waits for each answer
        dict(name="cascade_4x4096", kind="cascade", rows=4, vocab=4096, top_p=1.0),
        # the largest: an offline acceptance study over many positions with nucleus filtering
        dict(name="cascade_256x65536", kind="cascade", rows=256, vocab=65536, top_p=0.95),
        # the tiny fp32 decoder: launches and host work count, and the only 32-bit products
        model_case("tiny_decode", "decode", "tiny", "0/2/0", 4, 1, 2, 1, 33, 64),
        # the Ouro-1.4B shape, one user, greedy, at its best depth pair and the paper's prompt length
        model_case("ouro_decode", "decode", "ouro", "0/24/0", 4, 2, 3, 1, 512, 32),
        # the sampled Ouro setting (temperature 1, nucleus 0.95, depths 1 and 2) after a longer prompt; 8 of its blocks
        model_case("ouro_sampled", "decode", "ouro", "0/8/0", 4, 1, 2, 1, 1000, 24, temperature=1.0, top_p=0.95),
        # the whole Raven shape, 32 iterations, greedy, batch 1, at its best depth pair: the headline workload
        model_case("raven_decode", "decode", "raven", "2/4/2", 32, 16, 24, 1, 131, 8),
        # Raven width with early drafts and several users: trees of more than 16 branches (the wide launches)
        model_case("raven_tree", "decode", "raven", "1/2/1", 8, 1, 4, 3, 300, 8),
        # several users with long contexts on one handle: attention over the committed caches is most of the work
        model_case("long_batch", "decode", "ouro", "0/2/0", 4, 1, 2, 4, 6144, 16),
        # time to first token of the Ouro-1.4B shape
        model_case("ouro_prefill", "prefill", "ouro", "0/24/0", 4, 2, 3, 1, 512, 1),
        # the same at the Raven width, a ragged prompt, with prelude and coda blocks
        model_case("raven_prefill", "prefill", "raven", "1/2/1", 4, 1, 2, 1, 300, 1),
        # a long document: the prompt's causal attention grows with its square
        model_case("long_prefill", "prefill", "ouro", "0/2/0", 4, 1, 2, 1, 6000, 1),
        # the depth planner's measurement: readouts of a continuation at every depth
        model_case("ouro_readout", "readout", "ouro", "0/8/0", 4, 2, 3, 1, 200, 16),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cascade", "cascade", "prefill", "prefill", "readout", "decode", "decode", "decode"])
    if kind == "cascade":
        return dict(kind=kind, rows=log_int(rng, 1, 256), vocab=log_int(rng, 1000, 65536),
                    top_p=rng.choice([1.0, 0.95, 0.9, 0.7]))
    width = rng.choice(["tiny", "ragged", "ouro", "ouro", "raven"])
    big = width == "raven"
    pre, core, coda = {"tiny": (0, rng.randint(1, 3), 0), "ragged": (rng.randint(0, 1), rng.randint(1, 3), rng.randint(0, 1)),
                       "ouro": (0, rng.randint(1, 8), 0), "raven": (rng.randint(0, 1), rng.randint(1, 2), rng.randint(0, 1))}[width]
    R = rng.choice([3, 4, 4, 6, 8])
    d1 = rng.randint(1, R // 2)
    d2 = rng.choice([0] + list(range(d1 + 1, R)))
    prompt = log_int(rng, 2, 400 if big else 3000 if width == "ouro" else 1000)
    seqs, temperature, top_p, per_kernel, shared = 1, 0.0, 1.0, rng.random() < 0.25, False
    if kind == "decode":
        seqs = rng.choice([1, 1, 2, 3, 5])
        while seqs > 1 and seqs * worst_case_branches(R, d1, d2) > 64:
            seqs -= 1
        while worst_case_branches(R, d1, d2) > 64:
            d1, d2 = d1 + 1, 0
        shared = rng.random() < 0.15
        if rng.random() < 0.4:
            temperature, top_p = 1.0, rng.choice([1.0, 0.95, 0.9])
    elif worst_case_branches(R, d1, d2) > 64:
        d1, d2 = max(1, R // 2), 0
    tokens = 1 if kind == "prefill" else log_int(rng, 2, 12 if big else 24)
    return {k: v for k, v in model_case("", kind, width, "%d/%d/%d" % (pre, core, coda), R, d1, d2, seqs, prompt, tokens,
                                        temperature, top_p, per_kernel, shared).items() if k != "name"}


# ---------------------------------------------------------------------------------------------------------------------
# models and prompts
# ---------------------------------------------------------------------------------------------------------------------
LAYER = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "wg", "wu", "wd")


def spec_of(case):
    pre, core, coda = (int(x) for x in case["blocks"].split("/"))
    return types.SimpleNamespace(**WIDTHS[case["width"]], n_prelude=pre, n_core=core, n_coda=coda, rope_base=10000.0,
                                 rms_eps=1e-6, stacks=(("prelude", pre), ("core", core), ("coda", coda)))


def shape_of(sp, tensor):
    h, F = sp.hidden, sp.ffn
    return {"attn_norm": (h,), "ffn_norm": (h,), "wg": (F, h), "wu": (F, h), "wd": (h, F)}.get(tensor, (h, h))


@functools.lru_cache(maxsize=2)
def host_weights(width, blocks, R):
    """The model of a case in host memory, as a checkpoint loader hands it over: the same for every seed."""
    sp = spec_of(dict(width=width, blocks=blocks))
    h, F, V = sp.hidden, sp.ffn, sp.vocab
    g = torch.Generator(device=DEV).manual_seed(20)
    s = 0.02 * math.sqrt(h)                                   # standard deviation of a gate / up output
    inc = 0.02 * math.sqrt(F) * 0.64 * s * s                  # of one block's contribution at alpha = 1
    alpha = min(0.3, 1.0 / (inc * math.sqrt(sp.n_core) * R))
    out = {}

    def put(name, t):
        if sp.weight_dtype == "bf16":
            out[name] = t.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
        else:
            out[name] = t.cpu().numpy()

    def randn(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)

    embed = randn(V, h)
    put("embed", embed)
    put("final_norm", 1.0 + 0.1 * randn(h))
    if not sp.tied_head:
        perm = torch.randperm(V, generator=g, device=DEV)     # token t's successor is perm[t]
        head = torch.empty_like(embed)
        head[perm] = embed * (15.5 / (0.7 * h))
        put("head", head)
        del head
    del embed
    for stack, n in sp.stacks:
        for i in range(n):
            for t in LAYER:
                if t.endswith("norm"):
                    w = 1.0 + 0.1 * randn(h)
                else:
                    w = randn(*shape_of(sp, t)) * (math.sqrt(2.0 / h) if t in ("wq", "wk") else 0.02)
                    if t in ("wo", "wd"):
                        w *= alpha
                put("%s.%d.%s" % (stack, i, t), w)
    return out


def prompts_of(case, seed):
    """Prompts of a case: the first one has its full length, the others are a little shorter."""
    V = WIDTHS[case["width"]]["vocab"]
    rng = np.random.default_rng(seed)
    return [rng.integers(0, V, max(1, case["prompt"] - 7 * q)).astype(np.int32) for q in range(case["seqs"])]


def forced_of(case, seed):
    return np.random.default_rng(seed + 77).integers(0, WIDTHS[case["width"]]["vocab"], case["tokens"]).astype(np.int32)


def cascade_inputs(case, seed):
    """Readout logits at d1, d2 and R as a looped model gives them (deeper readouts closer to the last one), and keys."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = (case["rows"], case["vocab"])
    zR = 2.0 * torch.randn(*n, generator=g, device=DEV)
    z1 = zR + 0.6 * torch.randn(*n, generator=g, device=DEV)
    z2 = zR + 0.3 * torch.randn(*n, generator=g, device=DEV)
    pos = torch.randint(1, 8192, (case["rows"],), generator=g, device=DEV, dtype=torch.int32)
    keys = torch.stack([torch.arange(case["rows"], device=DEV, dtype=torch.int32), pos], 1).contiguous()
    return z1, z2, zR, keys


# ---------------------------------------------------------------------------------------------------------------------
# the measured calls
# ---------------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "cascade":
        return dict(case=case, inputs=cascade_inputs(case, seed))
    sp, prompts = spec_of(case), prompts_of(case, seed)
    dec = Decoder(sp, host_weights(case["width"], case["blocks"], case["R"]), R=case["R"], d1=case["d1"], d2=case["d2"],
                  temperature=case["temperature"], top_p=case["top_p"], seed=seed % 1000, max_seqs=case["seqs"],
                  max_ctx=case["prompt"] + case["tokens"] + 8, per_kernel=case["per_kernel"],
                  shared_prefix=case["shared_prefix"], device=DEV)
    if case["kind"] != "prefill":
        for q, ids in enumerate(prompts):
            dec.prefill(q, ids)
    return dict(case=case, dec=dec, prompts=prompts, forced=forced_of(case, seed))


def run(state):
    case = state["case"]
    if case["kind"] == "cascade":
        return run_cascade(*state["inputs"], temperature=1.0, top_p=case["top_p"], seed=2)
    dec = state["dec"]
    if case["kind"] == "prefill":
        first = dec.prefill(0, state["prompts"][0])
        logits, _ = dec.forced_readout(0, state["forced"])
        return dict(first=first, logits=logits)
    if case["kind"] == "readout":
        return dict(logits=dec.forced_readout(0, state["forced"])[0])
    for q in range(case["seqs"]):
        dec.rewind(q)
    tokens = dec.decode(case["tokens"])
    return dict(tokens=tokens, logits=np.stack([root_logits(dec, case, q) for q in range(case["seqs"])]))


def root_logits(dec, case, seq):
    """Readout at d1 of the newest committed token of a sequence (its root branch)."""
    for slot in range(dec.capacity()[0]):
        info, _ = dec.branch(slot, prefix=False)
        if info["active"] and info["seq"] == seq and info["parent"] == -1:
            for _ in range(case["d1"] - info["depth"]):       # a root that was resampled starts again at depth 0
                dec.decode_step()
            return dec.debug_readout(slot, case["d1"])
    raise RuntimeError("no root branch")


# ---------------------------------------------------------------------------------------------------------------------
# what the calls cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def work(case):
    """Every weight matrix is read once per pass over it: a prompt's rows go through one block application together, a
    generated token's depths follow each other.  LoopSpec decoding commits a token every d1 steps where drafts are
    accepted, with ceil(R / d1) branches in a pass; keys and values are read once per step, sequence and depth."""
    if case["kind"] == "cascade":
        n = case["rows"] * case["vocab"]
        return {"bytes": 4 * n * 5, "flops": 40 * n}
    sp = spec_of(case)
    e = 2 if sp.weight_dtype == "bf16" else 4
    h, F, V, R, n, k = sp.hidden, sp.ffn, sp.vocab, case["R"], case["prompt"], case["tokens"]
    block = 4 * h * h + 3 * h * F
    kv = 2 * h * e                                            # keys and values of one position in one block and depth

    def readouts():                                           # k positions on the vanilla schedule, read out everywhere
        apps = sp.n_prelude + R * (sp.n_core + sp.n_coda)
        return k * (apps * (block * e + n * kv) + R * h * V * e + R * V * 4), k * 2 * (apps * (block + 2 * n * h) + R * h * V)

    if case["kind"] == "readout":
        b, f = readouts()
        return {"bytes": b, "flops": f}
    if case["kind"] == "prefill":
        apps = sp.n_prelude + R * (sp.n_core + sp.n_coda)
        b, f = readouts()
        return {"bytes": b + apps * (block * e + n * kv) + h * V * e, "flops": f + 2 * apps * (block * n + n * n * h) + 2 * h * V}
    steps, rows = k * case["d1"], -(-R // case["d1"]) * case["seqs"]
    reads = 3 if case["d2"] else 2                            # readout depths: each is reached once per committed token
    bytes_ = steps * sp.n_core * (block * e + rows * n * kv) + k * (reads * (h * V + sp.n_coda * block) + sp.n_prelude * block) * e
    flops = 2 * k * case["seqs"] * (R * sp.n_core * (block + 2 * n * h) + reads * (h * V + sp.n_coda * block) + sp.n_prelude * block)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times what the calls are off from 64 bits: 3e-7 in fp32, 4e-4 with fp16 operands (largest entries about
    five times the rms).  The cascade's distributions are 1e-7 to 2e-5 off: a top-p cut or a race within rounding
    of a tie may move by one id: one such id is up to 1e-4 of a row's norm and 0.05 of its rms."""
    if case["kind"] == "cascade":
        return {"rel": 1e-4, "max": 0.2, "differ": 0.01}
    if WIDTHS[case["width"]]["weight_dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1.6e-3, "max": 1.6e-2}


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------
class Model64:
    """The looped forward pass in float64 with one cache of keys and values per (stack, depth, block)."""

    def __init__(self, case):
        self.sp, self.case, self.kv = spec_of(case), case, {}
        self.w = {k: torch.from_numpy(a.view(np.int16)).to(DEV).view(torch.bfloat16) if a.dtype == np.uint16 else
                  torch.from_numpy(a).to(DEV) for k, a in host_weights(case["width"], case["blocks"], case["R"]).items()}

    def norm(self, x, name):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + self.sp.rms_eps) * self.w[name].double()

    def lin(self, x, name):
        return x @ self.w[name].double().t()

    def rope(self, x, pos):
        half = self.sp.head_dim // 2
        ang = pos[:, None].double() * self.sp.rope_base ** (-2.0 * torch.arange(half, device=DEV).double() / self.sp.head_dim)
        c, s, a, b = ang.cos()[:, None], ang.sin()[:, None], x[..., :half], x[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def block(self, x, name, pos, space):
        H, dh = self.sp.n_heads, self.sp.head_dim
        y = self.norm(x, name + ".attn_norm")
        q, k, v = (self.lin(y, name + t).view(-1, H, dh) for t in (".wq", ".wk", ".wv"))
        q, k = self.rope(q, pos), self.rope(k, pos)
        if (space, name) in self.kv:
            k0, v0 = self.kv[(space, name)]
            k, v = torch.cat([k0, k]), torch.cat([v0, v])
        self.kv[(space, name)] = (k, v)
        kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
        outs = []
        for i in range(0, len(pos), 512):
            s = q[i:i + 512].permute(1, 0, 2).contiguous() @ kt / math.sqrt(dh)
            s = s.masked_fill(torch.arange(k.shape[0], device=DEV)[None, None] > pos[i:i + 512][None, :, None], -math.inf)
            outs.append((s.softmax(-1) @ vt).permute(1, 0, 2).reshape(-1, H * dh))
        x = x + self.lin(torch.cat(outs), name + ".wo")
        y = self.norm(x, name + ".ffn_norm")
        return x + self.lin(torch.nn.functional.silu(self.lin(y, name + ".wg")) * self.lin(y, name + ".wu"), name + ".wd")

    def advance(self, ids, first, depths):
        """Appends tokens at positions first..; the last position's logits at each of `depths`."""
        sp = self.sp
        pos = torch.arange(first, first + len(ids), device=DEV)
        x, got = self.w["embed"][torch.as_tensor(np.asarray(ids), device=DEV).long()].double(), {}
        for i in range(sp.n_prelude):
            x = self.block(x, "prelude.%d" % i, pos, "p")
        for r in range(1, self.case["R"] + 1):
            for i in range(sp.n_core):
                x = self.block(x, "core.%d" % i, pos, r)
            if r in depths:
                y = x
                for i in range(sp.n_coda):
                    y = self.block(y, "coda.%d" % i, pos, r)
                got[r] = self.lin(self.norm(y[-1:], "final_norm"), "embed" if sp.tied_head else "head")[0]
        return got


def exact(case, seed):
    if case["kind"] == "cascade":
        return exact_cascade(case, seed)
    R, every = case["R"], range(1, case["R"] + 1)
    if case["kind"] in ("prefill", "readout"):
        m, ids = Model64(case), prompts_of(case, seed)[0]
        got = m.advance(ids, 0, every)
        logits = []
        for i, t in enumerate(forced_of(case, seed)):
            z = m.advance([t], len(ids) + i, every)
            logits.append(torch.stack([z[r] for r in every]))
        logits = torch.stack(logits)
        return dict(first=int(got[R].argmax()), logits=logits) if case["kind"] == "prefill" else dict(logits=logits)
    if case["temperature"] > 0:                               # the draws are the library's own
        return None
    tokens, logits = [], []
    for ids in prompts_of(case, seed):
        m, row = Model64(case), []
        t = int(m.advance(ids, 0, (case["d1"], R))[R].argmax())
        for i in range(case["tokens"] + 1):
            z = m.advance([t], len(ids) + i, (case["d1"], R))
            t = int(z[R].argmax())
            row.append(t)
        tokens.append(row[:-1])
        logits.append(z[case["d1"]])
    return dict(tokens=np.array(tokens, np.int32), logits=torch.stack(logits))


EVENTS = dict(draft1=2, draft2=3, acc1=4, acc2=5, resample=6)


def uniforms(seed, seq, pos, event, n):
    """Top 24 bits (one value) or top 23 bits plus a half (a vocabulary) of Philox4x64-10 at counter (block, pos, event, 0)."""
    counter = ((EVENTS[event] << 128) | (int(pos) << 64)) - 1
    raw = np.random.Philox(counter=counter, key=(int(seq) << 64) | seed).random_raw(-(-n // 4) * 4)
    return float(raw[0] >> np.uint64(40)) * 2.0 ** -24 if n == 1 else ((raw[:n] >> np.uint64(41)).astype(np.float64) + 0.5) * 2.0 ** -23


def exact_cascade(case, seed):
    z1, z2, zR, keys = (t.cpu().numpy() for t in cascade_inputs(case, seed))
    V, out, q1s, q2s = case["vocab"], [], [], []

    def dist(z):
        z = z.astype(np.float64)
        p = np.exp(z - z.max())
        p /= p.sum()
        if case["top_p"] < 1.0:
            order = np.argsort(-p, kind="stable")
            c = np.cumsum(p[order])
            p[order[c - p[order] >= case["top_p"]]] = 0.0
            p /= p.sum()
        return p

    def minus(a, b):
        d = np.maximum(a - b, 0.0)
        return d / d.sum()

    for i, (seq, pos) in enumerate(keys):
        def race(w, event):
            return int(np.argmax(np.where(w > 0, w / -np.log(uniforms(2, seq, pos, event, V)), -np.inf)))

        q1, qt, p = dist(z1[i]), dist(z2[i]), dist(zR[i])
        x1 = race(q1, "draft1")
        gate, x2, q2 = qt[x1] < q1[x1], -1, np.zeros(V)
        if gate:
            q2 = minus(qt, q1)
            x2 = race(q2, "draft2")
        if uniforms(2, seq, pos, "acc1", 1) < min(1.0, p[x1] / q1[x1]):
            tok, src = x1, 1
        else:
            rho = minus(p, q1)
            if gate and uniforms(2, seq, pos, "acc2", 1) < min(1.0, rho[x2] / q2[x2]):
                tok, src = x2, 2
            else:
                tok, src = race(minus(rho, q2) if gate else rho, "resample"), 0
        out.append([tok, src, x1, int(gate), x2, 0])
        q1s.append(q1)
        q2s.append(q2)
    return np.array(out, np.int32), np.stack(q1s), np.stack(q2s)

"""Small 16-bit models whose readouts hang on the prompt's attention, and the
relative errors their tests allow.

The state's dimension 0 is the same at every token and block and makes up most
of its norm, so that the attention keeps its form from depth to depth; dimension
1 is set for token 0 alone.  Neither reaches the values, the FFN or the head."""
import numpy as np

import synth

# of a readout's norm: eight roundings to fp16 (2^-11 each); a row passes about four a block, which add up like a walk
REL = 8 * 2.0 ** -11


def f32(w, name):
    return synth.bf16_bits_to_f32(w[name]).copy()


def shaped(spec, noise, wv, wo):
    rng = np.random.default_rng(7)
    w = synth.make_weights(spec, seed=0)
    h = spec.hidden
    unit = np.sqrt(192.0 / h)

    def put(name, a):
        w[name] = synth.f32_to_bf16_bits(a.astype(np.float32))

    e = noise * rng.standard_normal((spec.vocab, h))
    e[:, 0], e[:, 1] = 8.0 / unit, 0.0
    put("embed", e)
    e = 0.3 * unit * rng.standard_normal((spec.vocab, h))
    e[:, :2] = 0.0
    put("head", e)
    for name in list(w):
        kind = name.rsplit(".", 1)[-1]
        if kind in ("wq", "wk"):
            put(name, 0.05 * unit * rng.standard_normal((h, h)))
        elif kind in ("wv", "wg", "wu"):
            a = wv * unit * rng.standard_normal((h, h)) if kind == "wv" else f32(w, name)
            a[:, :2] = 0.0
            put(name, a)
        elif kind in ("wo", "wd"):
            a = wo * unit * rng.standard_normal((h, h)) if kind == "wo" else f32(w, name)
            a[:2] = 0.0
            put(name, a)
    return w, put


def near_model(spec, nats=8.0):
    """Scores of `nats` times the mean cosine of RoPE's angles: near keys weigh most, by a power of the distance."""
    w, put = shaped(spec, noise=0.1, wv=0.15, wo=0.15)
    for name in list(w):
        if name.rsplit(".", 1)[-1] in ("wq", "wk"):
            a = f32(w, name)
            a[:, 0] = np.sqrt(nats / (np.sqrt(spec.head_dim) * spec.hidden))
            put(name, a)
    return w


SINK_NATS = 18.0


def sink_model(spec):
    """The other tokens' queries score token 0 SINK_NATS above the rest, and token 0's value is zero: the output is
    what the small weights add up to, which large values and output weights bring back to the state's size.  Token 0
    leads by the slow half of the rotations (rope_base far above the prompt's length)."""
    w, put = shaped(spec, noise=0.1, wv=3400.0, wo=36.0)
    h, dh = spec.hidden, spec.head_dim
    slow = np.arange(h) % (dh // 2) >= dh // 4
    ramp = np.tile(np.linspace(0.7, 1.3, dh), spec.n_heads) * slow
    s = np.sqrt(SINK_NATS * np.sqrt(dh) / (h * (ramp[:dh] ** 2).sum()))
    e = f32(w, "embed")
    e[0], e[0, 1] = 0.0, e[1, 0]
    put("embed", e)
    for name in list(w):
        kind = name.rsplit(".", 1)[-1]
        if kind in ("wq", "wk", "wv"):
            a = f32(w, name)
            if kind == "wv":
                a[:, 0] = 8000.0 / np.sqrt(h)
            else:
                a[slow] = 0.0
                a[:, 0 if kind == "wq" else 1] = s * ramp
            put(name, a)
    return w


def near_spec(H=1, dh=96, F=512, V=800):
    return synth.ModelSpec(H * dh, H, dh, F, V, 0, 1, 0, R=2, alpha=0.3)


def sink_spec(H=2, dh=96):
    return synth.ModelSpec(H * dh, H, dh, 256, 304, 0, 1, 0, R=2, alpha=0.3, rope_base=1e12)


def sink_prompt(spec, n=100):
    return [0] * 64 + [int(t) for t in np.random.default_rng(3).integers(1, spec.vocab, n)]


def readouts(lm, pr, tok, node=None):
    node = lm.extend(node or lm.prefill(pr), tok)
    return np.stack([lm.logits(node, r) for r in range(1, lm.spec.R + 1)])


def rel(a, b):
    return np.linalg.norm(a - b, axis=-1) / np.linalg.norm(b, axis=-1)


def readouts64(spec, w, ids):
    """The oracle's readouts [R, V] of the last of `ids`, for prompts too long for it: the same forward pass in float64
    on the GPU (core blocks only)."""
    import torch

    def t(name):
        a = w[name]
        return torch.from_numpy(synth.bf16_bits_to_f32(a) if a.dtype == np.uint16 else a).cuda().double()

    def norm(x, g):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + spec.rms_eps) * t(g)

    H, dh, T = spec.n_heads, spec.head_dim, len(ids)
    pos = torch.arange(T, device="cuda")
    ang = pos[:, None].double() * spec.rope_base ** (-2.0 * torch.arange(dh // 2, device="cuda").double() / dh)
    c, s = ang.cos()[:, None], ang.sin()[:, None]

    def rope(x):
        a, b = x[..., :dh // 2], x[..., dh // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    x, out = t("embed")[torch.as_tensor(np.asarray(ids)).long().cuda()], []
    for _ in range(spec.R):
        for i in range(spec.n_core):
            n = norm(x, f"core.{i}.attn_norm")
            q, k, v = ((n @ t(f"core.{i}.{m}").T).view(T, H, dh) for m in ("wq", "wk", "wv"))
            q, k, a = rope(q), rope(k), torch.empty_like(v)
            for h in range(H):
                kt, vh = k[:, h].T.contiguous(), v[:, h].contiguous()
                for r in range(0, T, 1024):
                    z = q[r:r + 1024, h].contiguous() @ kt / np.sqrt(dh)
                    a[r:r + 1024, h] = z.masked_fill(pos[None] > pos[r:r + 1024, None], -np.inf).softmax(-1) @ vh
            x = x + a.reshape(T, -1) @ t(f"core.{i}.wo").T
            n = norm(x, f"core.{i}.ffn_norm")
            x = x + (torch.nn.functional.silu(n @ t(f"core.{i}.wg").T) * (n @ t(f"core.{i}.wu").T)) @ t(f"core.{i}.wd").T
        out.append(norm(x[-1], "final_norm") @ t("head").T)
    return torch.stack(out).cpu().numpy()

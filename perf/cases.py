"""What a program does with this framework, as a list of measurable passes through its public entry points.

Four kinds of pass exist, one per thing a denoising program calls in its loop:

  stage   dp_stage_forward: one frame block through the layers one device owns, attending over the cached
          keys/values of the block processed before it (the cache is in the workspace when the call is made)
  embed   dp_embed_forward: latent frames -> tokens
  head    dp_head_forward (or dp_head_forward_static): tokens -> velocity in latent shape
  latent  the whole loop body on one device: embed -> stage -> cache hand-over -> head -> Euler update

Inputs are N(0, 1) tokens, latents and text and N(0, 0.02) weights, as everywhere in this repository, with two
differences that a trained model has and plain draws lack: gates of order one (otherwise no branch contributes
to the result) and q/k norm gains of 1.5 (attention that selects instead of averaging over all keys).
"""
import math

import torch

from paper_2505_21070_amd import binding as B
from paper_2505_21070_amd import synth

CHANNELS = 16                    # latent channels
T_NOW, T_NEIGHBOUR = 500.0, 625.0
LARGEST_FLOPS = 17e12            # of the largest listed case


def _stage(name, **kw):
    c = dict(name=name, path="stage", dtype="bf16", layout="out_in", n_layers=1, text_len=512, text_dim=4096,
             tok_h=30, tok_w=52, frames=4, cached=2, dim=1536, heads=12, head_dim=128, ffn=8960)
    c.update(kw)
    return c


def listed():
    return [
        # the largest single-device share in use: one 14B-shaped layer, 4 frames of 45 x 80 tokens and 2 cached
        _stage("layer_14b", dim=5120, heads=40, ffn=13824, tok_h=45, tok_w=80),
        # the same for the 1.3B shape: 4 frames of 30 x 52 tokens and 2 cached
        _stage("layer_1p3b"),
        # a video's first (longer) block, nothing cached yet, weights handed over [in, out]
        _stage("first_block", frames=5, cached=0, layout="in_out"),
        # blocks of 8 frames fed with 4 frames of context, 4 more cached: the longest sequences at this width
        _stage("extended_block", frames=12, cached=4),
        # one frame at a time (streaming, a video's ragged end): few tokens against full-size weights
        _stage("single_frame", frames=1),
        # head_dim 64, a narrower model, token counts that divide no tile, short text
        _stage("ragged_64", dim=1024, heads=16, head_dim=64, ffn=4096, tok_h=16, tok_w=21, frames=3,
               text_len=77, text_dim=1024, layout="in_out"),
        # a toy model: 216 tokens, 144 cached, text MLP in front; every kernel is short
        _stage("small", dim=256, heads=2, ffn=640, n_layers=2, text_len=40, text_dim=192, tok_h=6, tok_w=12,
               frames=3, layout="in_out"),
        # the smallest configuration, in fp32: 128 tokens, 64 cached, two layers
        _stage("tiny_f32", dtype="f32", dim=128, heads=2, head_dim=64, ffn=512, n_layers=2, text_len=16,
               text_dim=128, tok_h=8, tok_w=8, frames=2, cached=1, layout="in_out"),
        # fp32 at the 1.3B width, one frame and one cached: the run that a bf16 result is checked against
        _stage("frame_f32", dtype="f32", frames=1, cached=1, layout="in_out"),
        # the loop body of a whole denoiser on one device, in latent space (4 layers)
        _stage("latent_step", path="latent", n_layers=4),
        # the model's two ends: patch embedding of a block at the 1.3B shape, output head at the 14B shape
        dict(name="embed_1p3b", path="embed", dtype="bf16", dim=1536, tok_h=30, tok_w=52, frames=4),
        dict(name="head_14b", path="head", dtype="bf16", dim=5120, tok_h=45, tok_w=80, frames=4, static=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tokens(rng, even):
    """A frame's token grid; the bf16 stage takes grids of a multiple of 8 tokens."""
    while True:
        h, w = _log(rng, 5, 45), _log(rng, 6, 80)
        if w >= h and (not even or h * w % 8 == 0):
            return h, w


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        # fp32 runs at a tenth of the rate or less
        if w["flops"] <= (0.9 * LARGEST_FLOPS if c["dtype"] == "bf16" else 0.0098 * LARGEST_FLOPS):
            return c


def _draw(rng):
    path = rng.choices(("stage", "embed", "head", "latent"), (7, 1, 1, 1))[0]
    bf = path == "latent" or rng.random() < 0.8
    hd = rng.choice((64, 128, 128))
    top = (5120 if path != "latent" else 1536) if bf else 1536
    heads = max(1, _log(rng, 128, top) // hd)
    dim = heads * hd
    h, w = _tokens(rng, bf)
    c = dict(path=path, dtype="bf16" if bf else "f32", dim=dim, tok_h=h, tok_w=w, frames=rng.choice((1, 2, 3, 4, 4, 5, 8, 12)))
    if path == "embed":
        return c
    if path == "head":
        c["static"] = bool(rng.random() < 0.3)
        if c["static"] and _static_bytes(c) > (60 << 20):
            c["static"] = False
        return c
    ffn = 64 * max(2, int(dim * rng.uniform(2.0, 6.0) / 64))
    if rng.random() < 0.5:
        ffn = max(256, ffn // 256 * 256)
    c.update(n_layers=rng.choice((1, 1, 2)), heads=heads, head_dim=hd, ffn=ffn, cached=rng.choice((0, 1, 2, 2, 4)),
             text_len=_log(rng, 16, 512), text_dim=dim if rng.random() < 0.4 else 64 * _log(rng, 2, 64),
             layout="out_in" if bf and dim % 256 == 0 and ffn % 256 == 0 and rng.random() < 0.6 else "in_out")
    return c


def _static_bytes(c):
    E = 2 if c["dtype"] == "bf16" else 4
    S = (c["tok_h"] * c["tok_w"] * c["frames"] + 255) // 256 * 256
    return S * (c["dim"] * (4 + E) + 16 * CHANNELS) + 256 * c["dim"] * E + 80 * c["dim"] * 4


# ---------------------------------------------------------------------------------------------- inputs
def _cfg(c):
    cfg = dict(synth.DEFAULTS, dim=c["dim"], tok_h=c["tok_h"], tok_w=c["tok_w"], dtype=c["dtype"])
    if c["path"] in ("stage", "latent"):
        cfg.update(n_layers=c["n_layers"], n_heads=c["heads"], head_dim=c["head_dim"], ffn_dim=c["ffn"],
                   text_len=c["text_len"], text_dim=c["text_dim"], block_frames=c["frames"], cache_frames=c["cached"])
    return cfg


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _draws(c, seed):
    """Everything random of a case, in one fixed order, as device tensors: (weights, end weights, text, blocks, latent).
    Matrices are [in, out]."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    td, D = _dtype(c), c["dim"]

    def n(shape, scale=0.02, mean=0.0, dtype=td):
        t = torch.randn(shape, generator=g, dtype=torch.float32, device="cuda")
        return t.mul_(scale).add_(mean).to(dtype)

    S = c["frames"] * c["tok_h"] * c["tok_w"]
    fd = synth.DEFAULTS["freq_dim"]
    weights, ends, text, blocks, latent = None, None, None, None, None
    if c["path"] in ("stage", "latent"):
        stage_shapes, layer_shapes = synth.weight_shapes(_cfg(c))
        weights = {"stage": {k: n(s) for k, s in stage_shapes.items()}, "layers": []}
        for _ in range(c["n_layers"]):
            lw = {}
            for k, s in layer_shapes.items():
                lw[k] = n(s, mean=1.5 if k in ("gq", "gk", "cgq", "cgk") else 1.0 if k == "ln3_g" else 0.0)
                if k == "mod":
                    lw[k][2] += 1.0
                    lw[k][5] += 1.0
            weights["layers"].append(lw)
        text = n((c["text_len"], c["text_dim"]), 1.0)
        blocks = [n((S, D), 1.0) for _ in range(2)]
    if c["path"] != "stage":
        P = 4 * CHANNELS
        ends = dict(w_pe=n((P, D)), b_pe=n((D,)), m_head=n((2, D)), w_head=n((D, P)), b_head=n((P,)))
        if weights is not None:
            ends.update({k: weights["stage"][k] for k in ("wt1", "bt1", "wt2", "bt2")})
        else:
            ends.update(wt1=n((fd, D)), bt1=n((D,)), wt2=n((D, D)), bt2=n((D,)))
        if c["path"] != "head":
            latent = n((c["frames"], 2 * c["tok_h"], 2 * c["tok_w"], CHANNELS), 1.0, dtype=torch.float32)
        else:
            blocks = [n((S, D), 1.0)]
    return weights, ends, text, blocks, latent


def prepare(case, seed):
    c, cfg = case, _cfg(case)
    weights, ends, text, blocks, latent = _draws(c, seed)
    st = dict(case=c, ends=None)
    if weights is not None:
        conf = B.make_config(cfg, max_abs_frames=64, weight_layout=c["layout"])
        st["stage"] = B.Stage(conf, B.weights_out_in(weights) if c["layout"] == "out_in" else weights, text)
        # the neighbour, the later and noisier block, has been processed before and left its first frames' K/V
        if c["cached"]:
            k = min(c["cached"], c["frames"])
            st["stage"].forward(blocks[0], c["frames"], c["frames"], T_NEIGHBOUR)
            st["stage"].cache_update(0, k)
        st["x"] = blocks[1]
        st["out"] = torch.empty_like(blocks[1])
    if ends is not None:
        st["weights"], st["cfg"] = ends, cfg
        if c.get("static"):
            st["v"] = torch.empty((c["frames"], 2 * c["tok_h"], 2 * c["tok_w"], CHANNELS), dtype=torch.float32, device="cuda")
        else:
            st["ends"] = B.Ends(cfg, ends, CHANNELS, c["frames"])
        if c["path"] == "head":
            st["x"] = blocks[0]
        st["latent"] = latent
    return st


def run(state):
    c = state["case"]
    if c["path"] == "stage":
        return state["stage"].forward(state["x"], c["frames"], 0, T_NOW, out=state["out"])
    if c["path"] == "embed":
        return state["ends"].embed(state["latent"])
    if c["path"] == "head":
        if c["static"]:
            return B.head_forward_static(state["cfg"], state["weights"], CHANNELS, state["x"], T_NOW, c["frames"], state["v"])
        return state["ends"].head(state["x"], T_NOW, c["frames"])
    # one denoising step of one block; the latent is updated in place
    x = state["ends"].embed(state["latent"])
    y = state["stage"].forward(x, c["frames"], 0, T_NOW, out=state["out"])
    if c["cached"]:
        state["stage"].cache_update(0, min(c["cached"], c["frames"]))
    v = state["ends"].head(y, T_NOW, c["frames"])
    B.euler_step(state["latent"], v, 0.5, 0.48)
    return {"tokens": y, "velocity": v, "latent": state["latent"]}


# ---------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    c = case
    E, D = (2 if c["dtype"] == "bf16" else 4), c["dim"]
    S, P, fd = c["frames"] * c["tok_h"] * c["tok_w"], 4 * CHANNELS, synth.DEFAULTS["freq_dim"]
    by, fl = 0, 0
    if c["path"] in ("stage", "latent"):
        F, L, Lt = c["ffn"], c["n_layers"], c["text_len"]
        Nc = min(c["cached"], c["frames"]) * c["tok_h"] * c["tok_w"]
        by += L * E * (6 * D * D + 2 * D * F + 20 * D + F)          # the layer's weights
        by += E * (fd * D + D * D + 6 * D * D + 8 * D)              # timestep MLP and modulation head
        by += L * E * D * (2 * Nc + 2 * S + 2 * Lt) + 2 * E * S * D   # cached K/V in, own K/V kept, text K/V, tokens in and out
        fl += L * (2 * S * D * (6 * D + 2 * F) + 4 * S * (S + Nc + Lt) * D) + 2 * (fd * D + 7 * D * D)
    if c["path"] in ("embed", "latent"):
        by += E * (P * D + D) + 4 * S * P + E * S * D
        fl += 2 * S * P * D
    if c["path"] in ("head", "latent"):
        by += E * (P * D + fd * D + D * D + 4 * D) + 4 * S * P + E * S * D
        fl += 2 * S * P * D + 2 * (fd * D + D * D) + 8 * S * D
    if c["path"] == "latent":
        by += 3 * 4 * S * P                                        # Euler: two arrays in, one out
        fl += 2 * S * P
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # About four times the error measured against the same path in 64 bits: fp32 up to 1.3e-6; bf16 1.6e-3 to 2.3e-3
    # at the two ends, 1.7e-3 to 4.1e-3 for one or two layers, 5.7e-3 to 7.1e-3 for a whole loop body
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": {"embed": 1e-2, "head": 8e-3, "stage": 1.2e-2, "latent": 2.4e-2}[case["path"]]}


# ---------------------------------------------------------------------------------------------- 64 bits
def _f64(t):
    return t.double()


def _time_embedding(w, t):
    fd = w["wt1"].shape[0]
    half = fd // 2
    om = torch.pow(torch.tensor(10000.0, dtype=torch.float64, device="cuda"),
                   -torch.arange(half, dtype=torch.float64, device="cuda") / half)
    tau = torch.cat([torch.cos(t * om), torch.sin(t * om)])[None, :]
    silu = torch.nn.functional.silu
    return silu(tau @ _f64(w["wt1"]) + _f64(w["bt1"])) @ _f64(w["wt2"]) + _f64(w["bt2"])


def _norm(x, eps):
    m = x.mean(1, keepdim=True)
    return (x - m) * torch.rsqrt((x - m).square().mean(1, keepdim=True) + eps)


def _rms(x, g, eps):
    return x * torch.rsqrt(x.square().mean(1, keepdim=True) + eps) * _f64(g)


def _rope(x, c, frame0, theta):
    S, hd = x.shape[0], c["head_dim"]
    half, sp = hd // 2, hd // 6
    pairs = (half - 2 * sp, sp, sp)
    tok = c["tok_h"] * c["tok_w"]
    s = torch.arange(S, device="cuda")
    pos = (frame0 + s // tok, s % tok // c["tok_w"], s % tok % c["tok_w"])
    ang = torch.cat([p.double()[:, None] * torch.pow(torch.tensor(theta, dtype=torch.float64, device="cuda"),
                     -torch.arange(n, dtype=torch.float64, device="cuda") / n)[None, :] for p, n in zip(pos, pairs) if n], dim=1)
    co, si = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    v = x.reshape(S, c["heads"], half, 2)
    a, b = v[..., 0], v[..., 1]
    return torch.stack([a * co - b * si, a * si + b * co], dim=-1).reshape(S, -1)


def _attend(q, k, v, c):
    hd, out = c["head_dim"], torch.empty_like(q)
    for h in range(c["heads"]):
        cols = slice(h * hd, (h + 1) * hd)
        kt, vh = k[:, cols].t().contiguous(), v[:, cols].contiguous()
        for r in range(0, q.shape[0], 2048):
            p = torch.softmax(q[r:r + 2048, cols].contiguous() @ kt / math.sqrt(hd), dim=1)
            out[r:r + 2048, cols] = p @ vh
    return out


def _gelu(x):
    return torch.nn.functional.gelu(x, approximate="tanh")


def _layers(c, weights, text, x, frame0, t, cache):
    """All layers on one block; cache: per layer (K, V) or None.  Returns the result and each layer's own (K, V)."""
    eps, theta = synth.DEFAULTS["eps"], synth.DEFAULTS["rope_theta"]
    w = weights["stage"]
    e0 = (torch.nn.functional.silu(_time_embedding(w, t)) @ _f64(w["wm"]) + _f64(w["bm"])).reshape(6, -1)
    ctx = _f64(text)
    if "wx1" in w:
        ctx = _gelu(ctx @ _f64(w["wx1"]) + _f64(w["bx1"])) @ _f64(w["wx2"]) + _f64(w["bx2"])
    own = []
    for l, lw in enumerate(weights["layers"]):
        def lin(a, m, b):
            return a @ _f64(lw[m]) + _f64(lw[b])
        sh1, sc1, g1, sh2, sc2, g2 = _f64(lw["mod"]) + e0
        hn = _norm(x, eps) * (1 + sc1) + sh1
        q = _rope(_rms(lin(hn, "wq", "bq"), lw["gq"], eps), c, frame0, theta)
        k = _rope(_rms(lin(hn, "wk", "bk"), lw["gk"], eps), c, frame0, theta)
        v = lin(hn, "wv", "bv")
        own.append((k, v))
        ka, va = (k, v) if cache is None else (torch.cat([cache[l][0], k]), torch.cat([cache[l][1], v]))
        x = x + g1 * lin(_attend(q, ka, va, c), "wo", "bo")
        u = _norm(x, eps) * _f64(lw["ln3_g"]) + _f64(lw["ln3_b"])
        cq = _rms(lin(u, "cwq", "cbq"), lw["cgq"], eps)
        ck = _rms(lin(ctx, "cwk", "cbk"), lw["cgk"], eps)
        x = x + lin(_attend(cq, ck, lin(ctx, "cwv", "cbv"), c), "cwo", "cbo")
        f = _norm(x, eps) * (1 + sc2) + sh2
        x = x + g2 * lin(_gelu(lin(f, "w1", "b1")), "w2", "b2")
    return x, own


def _embed64(c, ends, latent):
    F, h, w = c["frames"], c["tok_h"], c["tok_w"]
    p = latent.double().reshape(F, h, 2, w, 2, CHANNELS).permute(0, 1, 3, 2, 4, 5).reshape(F * h * w, 4 * CHANNELS)
    return p @ _f64(ends["w_pe"]) + _f64(ends["b_pe"])


def _head64(c, ends, x, t):
    F, h, w = c["frames"], c["tok_h"], c["tok_w"]
    shift, scale = _f64(ends["m_head"]) + _time_embedding(ends, t)
    o = (_norm(x, synth.DEFAULTS["eps"]) * (1 + scale) + shift) @ _f64(ends["w_head"]) + _f64(ends["b_head"])
    return o.reshape(F, h, w, 2, 2, CHANNELS).permute(0, 1, 3, 2, 4, 5).reshape(F, 2 * h, 2 * w, CHANNELS)


def exact(case, seed):
    c = case
    weights, ends, text, blocks, latent = _draws(c, seed)
    if c["path"] == "embed":
        return _embed64(c, ends, latent)
    if c["path"] == "head":
        return _head64(c, ends, _f64(blocks[0]), T_NOW)
    cache = None
    if c["cached"]:
        n = min(c["cached"], c["frames"]) * c["tok_h"] * c["tok_w"]
        _, own = _layers(c, weights, text, _f64(blocks[0]), c["frames"], T_NEIGHBOUR, None)
        cache = [(k[:n].clone(), v[:n].clone()) for k, v in own]
    if c["path"] == "stage":
        return _layers(c, weights, text, _f64(blocks[1]), 0, T_NOW, cache)[0]
    y, _ = _layers(c, weights, text, _embed64(c, ends, latent), 0, T_NOW, cache)
    v = _head64(c, ends, y, T_NOW)
    return {"tokens": y, "velocity": v, "latent": latent.double() + (0.48 - 0.5) * v}

"""The workloads that this framework's speed is judged by.

Each case is one call sequence through the public entry points: a transformer
evaluation (``cs_velocity``), a whole candidate rollout (``run_rollout``:
rollout init, every denoise step with its cache decision, latents, scores) or
the scoring of finished latents (``cs_score_noalloc``).  Model shapes are the
registry's (``paper_2607_23159_amd.synth.MODELS``); the drawn cases keep their
widths and vary tokens, depth, batch, text length, mode and data type.

A block of a network is a one- or two-block model: ``cs_velocity`` is the entry
point that takes one.  Weights are drawn at the scale that keeps activations
at order one through the layers (matrices N(0, 1/fan_in), norm gains around
one, gates around one), so that every branch reaches the output.

Rollouts in bf16 use the modes whose schedule is fixed by the step number, so
that a rounding cannot flip a decision; the fp32 rollouts use the drift rule.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2607_23159_amd import binding as B
from paper_2607_23159_amd import search, synth

BF16, FP32 = synth.DTYPE_BF16, synth.DTYPE_FP32
MODES = {"off": synth.CACHE_OFF, "adaptive": synth.CACHE_ADAPTIVE, "static": synth.CACHE_STATIC,
         "pab": synth.CACHE_PAB}


# ------------------------------------------------------------------- cases
def _velocity(name, model, n, **kw):
    return dict(name=name, kind="velocity", model=model, n=n, **kw)


def _rollout(name, model, n, steps, mode, **kw):
    return dict(name=name, kind="rollout", model=model, n=n, steps=steps, mode=mode, **kw)


def listed():
    return [
        # Ranking a finished batch of eight 480p latents: two launches, the
        # shortest call of the library.
        dict(name="score_8x480p", kind="score", n=8, numel=synth.MODELS["wan13b"].latent_numel),
        # The smallest whole search step: the tiny workload as its
        # configuration states it (fp32, 4 seeds, 10 steps, tau = 0.1).
        # Nothing but latency: launches, the per-step read-back, allocations.
        _rollout("tiny_rollout_fp32", "tiny", 4, 10, "adaptive", fp32=True),
        # A small odd geometry (297 tokens, 19 text tokens, 64-wide heads) in
        # bf16: no tile size divides it.
        _velocity("ragged_bf16_n3", "ragged", 3),
        # Wan2.1-1.3B widths on a thumbnail latent, one stream: a latency-bound
        # evaluation at full width.
        _velocity("mid13b_n1", "wan_mid", 1),
        # The same widths in fp32, the type used to check bf16 results.
        _velocity("mid13b_fp32_n2", "wan_mid", 2, fp32=True),
        # Attention-output broadcasting (the second reuse engine), short
        # latents, four seeds.
        _rollout("mid13b_pab", "wan_mid", 4, 10, "pab"),
        # Wan2.1-14B widths, a small batch.
        _velocity("mid14b_n4", "wan14b_mid", 4),
        # A whole guided search over one-frame previews with the complete
        # 30-block 1.3B model: 4 seeds x 2 branches of 1,560 tokens.
        _rollout("frame13b_cfg_rollout", "wan13b", 4, 10, "static", lat_f=1, branches=2, static_k=4),
        # One 1.3B block at the full 32,760 tokens, one stream (a committed
        # winner, a single seed).
        _velocity("block13b_n1", "wan13b_block1", 1),
        # The same with the eight seeds of the headline search in one batch.
        _velocity("block13b_n8", "wan13b_block1", 8),
        # One Wan2.2-5B block at 27,280 tokens (ragged last tiles), four seeds.
        _velocity("block5b_n4", "wan5b", 4, blocks=1),
        # A complete 30-block evaluation of one 480p video.
        _velocity("full13b_n1", "wan13b", 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_grid(rng, lo, hi):
    """Odd and even patch grids with about lo..hi tokens."""
    tokens = _log_int(rng, lo, hi)
    f = min(rng.randint(1, 21), max(1, tokens // 32))
    hw = max(12, tokens // f)
    h = max(3, int(round(math.sqrt(hw) * rng.uniform(0.6, 1.0))))
    w = max(3, hw // h)
    return f, 2 * h, 2 * w


def draw(rng):
    kind = rng.choice(["score", "velocity", "velocity", "velocity", "fp32", "small", "rollout", "rollout"])
    if kind == "score":
        f, h, w = _draw_grid(rng, 256, 32760)
        return dict(kind="score", n=_log_int(rng, 1, 32), numel=16 * f * h * w)
    if kind == "velocity":
        model = rng.choice(["wan_mid", "wan_mid", "wan5b_mid", "wan14b_mid"])
        # at 14B width a full-length stream of one block costs 3x the 1.3B one
        f, h, w = _draw_grid(rng, 200, {"wan_mid": 32760, "wan5b_mid": 27280, "wan14b_mid": 12000}[model])
        tokens = f * h * w // 4
        n = min(8, max(1, 262080 // tokens), _log_int(rng, 1, 8))
        blocks = rng.choice([1, 2]) if n * tokens < 65536 else 1
        return dict(kind="velocity", model=model, n=n, blocks=blocks, lat_f=f, lat_h=h, lat_w=w,
                    text_len=rng.choice([512, 512, 226, 77]))
    if kind == "fp32":
        f, h, w = _draw_grid(rng, 60, 1200)
        return dict(kind="velocity", model=rng.choice(["tiny", "ragged", "wan_mid"]), n=rng.randint(1, 4),
                    lat_f=f, lat_h=h, lat_w=w, fp32=True)
    if kind == "small":
        f, h, w = _draw_grid(rng, 60, 4000)
        return dict(kind="velocity", model=rng.choice(["tiny", "ragged"]), n=_log_int(rng, 1, 16),
                    blocks=rng.randint(1, 4), lat_f=f, lat_h=h, lat_w=w, text_len=rng.randint(8, 300))
    branches = rng.choice([1, 2])
    if rng.random() < 0.4:
        f, h, w = _draw_grid(rng, 60, 600)
        return dict(kind="rollout", model=rng.choice(["tiny", "ragged"]), n=rng.randint(1, 12),
                    steps=rng.randint(4, 16), mode="adaptive", branches=branches, lat_f=f, lat_h=h, lat_w=w,
                    fp32=True)
    f, h, w = _draw_grid(rng, 200, 3200)
    return dict(kind="rollout", model="wan_mid", n=rng.randint(1, 8), steps=rng.randint(4, 12),
                mode=rng.choice(["static", "pab", "off"]), static_k=rng.randint(2, 5), branches=branches,
                blocks=rng.randint(1, 6), lat_f=f, lat_h=h, lat_w=w)


# ------------------------------------------------------------------ inputs
def _cfg(case):
    m = synth.MODELS[case["model"]]
    keys = {"blocks": "n_blocks", "lat_f": "lat_f", "lat_h": "lat_h", "lat_w": "lat_w", "text_len": "text_len"}
    m = dataclasses.replace(m, **{f: case[k] for k, f in keys.items() if k in case})
    return m.with_dtype(FP32 if case.get("fp32") else BF16)


def _roll(case):
    return synth.RolloutCfg(n_cand=case["n"], n_steps=case["steps"], n_branch=case.get("branches", 1),
                            k_warm=1, k_cool=1, tau=0.1, mode=MODES[case["mode"]],
                            static_k=case.get("static_k", 2))


def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000 + salt)


def _weights(m, seed):
    """Flat fp32 weights on the device in ``synth.weight_spec`` order."""
    spec = synth.weight_spec(m)
    flat = torch.randn(synth.weight_count(m), generator=_gen(seed, 1), device="cuda")
    off = 0
    for name, shape, kind in spec:
        v = flat[off:off + math.prod(shape)].view(shape)
        off += v.numel()
        if kind == "one":
            v.mul_(0.1).add_(1.0)
        elif kind == "gate":
            v.mul_(0.1)
            v[2].add_(1.0)
            v[5].add_(1.0)
        elif name.endswith("_w"):
            v.mul_(shape[1] ** -0.5)
        else:
            v.mul_(0.1)
    return flat


def _contexts(m, seed, n):
    return [torch.randn(m.text_len, m.text_dim, generator=_gen(seed, 2 + b), device="cuda") for b in range(n)]


def _latents(m, seed, n):
    return torch.randn((n,) + m.latent_shape, generator=_gen(seed, 5), device="cuda")


def _timestep(seed):
    return 0.05 + 0.9 * ((int(seed) * 0.6180339887) % 1.0)


class _Model:
    """A model handle, given back with the object that holds it."""

    def __init__(self, m, weights):
        self.cfg = m
        self.h = B.cs_model_init(B.model_desc(m), weights, weights.numel())

    def __del__(self):
        if getattr(self, "h", 0):
            B.cs_model_free(self.h)
            self.h = 0


def prepare(case, seed):
    if case["kind"] == "score":
        x = torch.randn(case["n"], case["numel"], generator=_gen(seed, 5), device="cuda")
        w = torch.randn(case["numel"], generator=_gen(seed, 6), device="cuda")
        return dict(case=case, x=x, w=w)
    m = _cfg(case)
    state = dict(case=case, model=_Model(m, _weights(m, seed)))
    x = _latents(m, seed, case["n"])
    if case["kind"] == "velocity":
        return dict(state, x=x, ctx=_contexts(m, seed, 1)[0], t=_timestep(seed))
    r = _roll(case)
    ctx = _contexts(m, seed, r.n_branch)
    w = torch.randn(m.latent_numel, generator=_gen(seed, 6), device="cuda")
    wl = synth.Workload("case", m, r, np.empty(0, np.float32), [c.cpu().numpy() for c in ctx], x.cpu().numpy(),
                        w.cpu().numpy(), synth.timestep_grid(r.n_steps))
    return dict(state, wl=wl, inputs=search.Inputs(wl))


def run(state):
    case = state["case"]
    if case["kind"] == "score":
        x, w = state["x"], state["w"]
        scores = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
        B.cs_score_noalloc(x, w, x.shape[0], x.shape[1], scores)
        return scores
    if case["kind"] == "velocity":
        x = state["x"]
        v = torch.empty_like(x)
        B.cs_velocity(state["model"].h, x, x.shape[0], state["t"], state["ctx"], v)
        return v
    g = search.run_rollout(state["model"], state["wl"], state["inputs"])
    out = {"latents": g.latents, "masks": g.masks}
    if case.get("fp32"):
        # In bf16 the scores are compared through the latents they project:
        # a random sum of 1e5 terms may lie near zero, where its relative
        # error says nothing.
        out["scores"] = g.scores
    return out


# -------------------------------------------------------------------- work
def _eval_flops(m):
    """One transformer call on one latent, text keys and values aside."""
    L, d = m.tokens, m.hidden
    per_block = 2 * L * (6 * d * d + 2 * d * m.ffn) + 4 * L * L * d + 4 * L * m.text_len * d
    return m.n_blocks * per_block + 4 * L * d * m.patch_dim


def _text_flops(m):
    d = m.hidden
    return 2 * m.text_len * (m.text_dim * d + d * d + 2 * m.n_blocks * d * d)


def _computed_steps(r):
    """Steps whose transformer calls cannot be left out; the drift rule
    computes four calls of ten on the tiny workload."""
    if r.mode in (synth.CACHE_OFF, synth.CACHE_PAB):
        return r.n_steps
    if r.mode == synth.CACHE_ADAPTIVE:
        return max(2, round(0.4 * r.n_steps))
    return sum(s <= r.k_warm or s > r.n_steps - r.k_cool or (s - r.k_warm) % r.static_k == 0
               for s in range(1, r.n_steps + 1))


def work(case):
    if case["kind"] == "score":
        return {"bytes": 4 * case["numel"] * (case["n"] + 1) + 8 * case["n"],
                "flops": 2 * case["numel"] * case["n"]}
    m = _cfg(case)
    weights = synth.weight_count(m) * (4 if m.dtype == FP32 else 2)
    text = 4 * m.text_len * m.text_dim
    lat = 4 * case["n"] * m.latent_numel
    if case["kind"] == "velocity":
        return {"bytes": weights + text + 2 * lat, "flops": case["n"] * _eval_flops(m) + _text_flops(m)}
    r = _roll(case)
    k = _computed_steps(r)
    flops = k * r.n_cand * r.n_branch * _eval_flops(m)
    if r.mode == synth.CACHE_PAB:
        # reused attentions: what the broadcast schedule leaves of them
        def computes(rng):
            return sum(s <= r.k_warm or s > r.n_steps - r.k_cool or (s - r.k_warm) % rng == 0
                       for s in range(1, r.n_steps + 1))
        L, d = m.tokens, m.hidden
        per_self = m.n_blocks * (2 * L * 4 * d * d + 4 * L * L * d)
        per_cross = m.n_blocks * (2 * L * 2 * d * d + 4 * L * m.text_len * d)
        flops -= r.n_cand * r.n_branch * ((r.n_steps - computes(r.pab_self)) * per_self +
                                          (r.n_steps - computes(r.pab_cross)) * per_cross)
    return {"bytes": k * weights + r.n_branch * text + 2 * lat * r.n_steps,
            "flops": flops + r.n_branch * _text_flops(m)}


# --------------------------------------------------------------- tolerance
def tolerance(case):
    """About four times the distance measured to the 64-bit result: 3e-16 for
    the fp64 sums of the scores (a sum in another order moves a few of their
    last bits), 1.5e-6 in fp32, 5.5e-3 for a bf16 evaluation and 8e-3 for the
    latents of a guided bf16 rollout."""
    if case["kind"] == "score":
        return {"rel": 1e-14}
    if case.get("fp32"):
        return {"rel": 8e-6}
    return {"rel": 2e-2 if case["kind"] == "velocity" else 3e-2}


# ------------------------------------------------------ 64-bit computation
def _ln(z):
    z = z - z.mean(-1, keepdim=True)
    return z / torch.sqrt((z * z).mean(-1, keepdim=True) + 1e-6)


def _rms(z, g):
    return z / torch.sqrt((z * z).mean(-1, keepdim=True) + 1e-6) * g


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x * x * x)))


def _lin(x, w, b):
    return torch.addmm(b, x, w.t())


class _Exact:
    """The network in 64 bits on the device, one stream at a time."""

    def __init__(self, m, flat):
        self.m = m
        self.w, off = {}, 0
        for name, shape, _ in synth.weight_spec(m):
            self.w[name] = flat[off:off + math.prod(shape)].view(shape)
            off += math.prod(shape)
        f, h, w = m.grid
        half = m.head_dim // 2
        n_h = n_w = m.head_dim // 6
        n_f = half - n_h - n_w
        axes = torch.meshgrid(*(torch.arange(k, device="cuda", dtype=torch.float64) for k in (f, h, w)),
                              indexing="ij")
        ang = torch.cat([a.reshape(-1, 1) * 10000.0 ** (-torch.arange(n, device="cuda", dtype=torch.float64) / n)
                         for a, n in zip(axes, (n_f, n_h, n_w))], dim=1)
        self.cos, self.sin = ang.cos()[:, None], ang.sin()[:, None]

    def p(self, name):
        return self.w[name].double().reshape(-1) if self.w[name].shape[0] == 1 else self.w[name].double()

    def rope(self, x):
        y = x.view(x.shape[0], self.m.heads, -1, 2)
        a, b = y[..., 0], y[..., 1]
        return torch.stack([a * self.cos - b * self.sin, a * self.sin + b * self.cos], -1).reshape(x.shape)

    def attention(self, q, k, v):
        dh = self.m.head_dim
        out = torch.empty_like(q)
        rows = max(64, (1 << 28) // k.shape[0])
        for h in range(self.m.heads):
            c = slice(h * dh, (h + 1) * dh)
            kt, vh = (k[:, c] / math.sqrt(dh)).t().contiguous(), v[:, c].contiguous()
            for i in range(0, q.shape[0], rows):
                out[i:i + rows, c] = torch.softmax(q[i:i + rows, c].contiguous() @ kt, -1) @ vh
        return out

    def text(self, ctx):
        h = _gelu(_lin(ctx.double(), self.p("text1_w"), self.p("text1_b")))
        return _lin(h, self.p("text2_w"), self.p("text2_b"))

    def velocity(self, x, t, emb, stored=None, reuse=(False, False)):
        """``stored``: per-block [self, cross] attention outputs, read where
        ``reuse`` says so and written otherwise."""
        m, d = self.m, self.m.hidden
        c, f, h, w = m.latent_shape
        om = 10000.0 ** (-torch.arange(128, device="cuda", dtype=torch.float64) / 128)
        arg = (1000.0 * float(np.float32(t)) * om)[None]
        s = torch.cat([arg.cos(), arg.sin()], 1)
        silu = torch.nn.functional.silu
        e = _lin(silu(_lin(s, self.p("time1_w"), self.p("time1_b"))), self.p("time2_w"), self.p("time2_b"))
        m6 = _lin(silu(e), self.p("mod_w"), self.p("mod_b")).view(6, d)
        z = x.double().view(c, f, h // 2, 2, w // 2, 2).permute(1, 2, 4, 0, 3, 5).reshape(m.tokens, -1)
        z = _lin(z, self.p("patch_w"), self.p("patch_b"))
        for j in range(m.n_blocks):
            b = f"blk{j}."
            sh1, sc1, g1, sh2, sc2, g2 = m6 + self.p(b + "mod")
            if reuse[0]:
                y = stored[j][0]
            else:
                qkv = _lin(_ln(z) * (1 + sc1) + sh1, self.p(b + "qkv_w"), self.p(b + "qkv_b"))
                q, k, v = qkv.split(d, 1)
                y = self.attention(self.rope(_rms(q, self.p(b + "q_gain"))),
                                   self.rope(_rms(k, self.p(b + "k_gain"))), v)
                y = _lin(y, self.p(b + "o_w"), self.p(b + "o_b"))
            z = z + g1 * y
            if reuse[1]:
                yc = stored[j][1]
            else:
                u = _ln(z) * self.p(b + "ca_ln_g") + self.p(b + "ca_ln_b")
                q = _rms(_lin(u, self.p(b + "caq_w"), self.p(b + "caq_b")), self.p(b + "caq_gain"))
                k = _rms(_lin(emb, self.p(b + "cak_w"), self.p(b + "cak_b")), self.p(b + "cak_gain"))
                yc = self.attention(q, k, _lin(emb, self.p(b + "cav_w"), self.p(b + "cav_b")))
                yc = _lin(yc, self.p(b + "cao_w"), self.p(b + "cao_b"))
            z = z + yc
            if stored is not None:
                stored[j] = [y, yc]
            u = _lin(_ln(z) * (1 + sc2) + sh2, self.p(b + "ffn1_w"), self.p(b + "ffn1_b"))
            z = z + g2 * _lin(_gelu(u), self.p(b + "ffn2_w"), self.p(b + "ffn2_b"))
        sh, sc = e + self.p("head_mod")
        y = _lin(_ln(z) * (1 + sc) + sh, self.p("head_w"), self.p("head_b"))
        return y.view(f, h // 2, w // 2, c, 2, 2).permute(3, 0, 1, 4, 2, 5).reshape(c, f, h, w)


def _exact_rollout(net, r, x, ctx, w, grid):
    embs = [net.text(c) for c in ctx]
    x = x.double()
    shape = (r.n_cand, r.n_branch)
    ref, delta = {}, {}
    acc = np.zeros(shape)
    stored = {(i, b): [None] * net.m.n_blocks for i in range(shape[0]) for b in range(shape[1])}
    masks = np.zeros((r.n_steps, r.n_cand * r.n_branch), np.uint8)
    for k in range(1, r.n_steps + 1):
        t0, dt = grid[k - 1], float(grid[k]) - float(grid[k - 1])
        window = k <= r.k_warm or k > r.n_steps - r.k_cool
        for i in range(r.n_cand):
            v = []
            for b in range(r.n_branch):
                s = (i, b)
                reuse = (False, False)
                if r.mode == synth.CACHE_PAB:
                    compute = True
                    reuse = tuple(not window and k > 1 and (k - r.k_warm) % g != 0
                                  for g in (r.pab_self, r.pab_cross))
                elif window or r.mode == synth.CACHE_OFF or s not in ref:
                    compute = True
                elif r.mode == synth.CACHE_STATIC:
                    compute = (k - r.k_warm) % r.static_k == 0
                else:
                    acc[s] += ((x[i] - ref[s]).norm() / ref[s].norm()).item()
                    compute = acc[s] > float(np.float32(r.tau))
                if compute:
                    keep = stored[s] if r.mode == synth.CACHE_PAB else None
                    v.append(net.velocity(x[i], t0, embs[b], keep, reuse))
                    ref[s], delta[s], acc[s] = x[i].clone(), v[b] - x[i], 0.0
                    masks[k - 1, i * r.n_branch + b] = 1
                else:
                    v.append(x[i] + delta[s])
            vt = v[0] if r.n_branch == 1 else v[1] + r.guidance * (v[0] - v[1])
            x[i] += dt * vt
    scores = (x.reshape(r.n_cand, -1) @ w.double()) / math.sqrt(w.numel())
    out = {"latents": x.cpu().numpy(), "masks": masks}
    if net.m.dtype == FP32:
        out["scores"] = scores.cpu().numpy()
    return out


def exact(case, seed):
    if case["kind"] == "score":
        s = prepare(case, seed)
        # the products of fp32 values and their sum in 64 bits
        return (s["x"].double() @ s["w"].double()) / math.sqrt(case["numel"])
    # about what a 64-bit matrix product does in 20 seconds
    if work(case)["flops"] > 4e14:
        return None
    m = _cfg(case)
    net = _Exact(m, _weights(m, seed))
    x = _latents(m, seed, case["n"])
    if case["kind"] == "velocity":
        emb = net.text(_contexts(m, seed, 1)[0])
        t = _timestep(seed)
        return torch.stack([net.velocity(x[i], t, emb) for i in range(case["n"])])
    r = _roll(case)
    w = torch.randn(m.latent_numel, generator=_gen(seed, 6), device="cuda")
    return _exact_rollout(net, r, x, _contexts(m, seed, r.n_branch), w, synth.timestep_grid(r.n_steps))

"""Workloads of the denoising hot path, as a user's program runs them through the Python binding.

Kinds of work:
  forward  one noise-predictor call: the dominant cost of every denoising step
  run      a whole reuse-then-predict run, one predictor call per step or one per cycle
  attn     the stand-alone 3D attention call
  linear   one projection of a layer
  update   the bookkeeping of one step: scheduler update with its four sums, relative MAE against another run

`listed()` names one case per situation; `draw()` gives others of the same ranges.  Inputs and weights are
Gaussian, made on the GPU from the seed.  Matrices are N(0, 1/fan_in) and the gates of every layer are 1 plus noise,
so that logits, activations and gates are of order one and every sub-layer counts, as in a trained network.
"""
import math

import torch

from paper_2505_14741_amd import binding as B
from paper_2505_14741_amd import inputs as I


def listed():
    net = {"layers": 30, "batch": 1, "dtype": "bf16"}
    return [
        # the small fp32 network: 8 DDIM steps, 2 warm-up steps, reuse window 2; every launch is tiny, latency counts
        {"name": "tiny_run", "kind": "run", "base": "tiny", "layers": 2, "frames": 2, "rows": 8, "cols": 8, "text": 0,
         "dtype": "f32", "steps": 8, "warmup": 2, "window": 2, "batched": False},
        # the whole 30-layer bf16 network on few tokens: a preview resolution; every weight is read for 112 tokens
        dict(net, name="reduced_step", kind="forward", frames=2, rows=6, cols=8, text=16),
        # the same network, step-batched: warm-up, then two cycles of four steps in one predictor call each
        {"name": "reduced_batched_run", "kind": "run", "base": "reduced", "layers": 30, "frames": 2, "rows": 6, "cols": 8,
         "text": 16, "dtype": "bf16", "steps": 9, "warmup": 1, "window": 4, "batched": True},
        # fp32 at the real width: what one runs to check a bf16 result
        dict(net, name="f32_step", kind="forward", layers=2, frames=2, rows=6, cols=8, text=16, dtype="f32"),
        # one block on 4290 video + 226 text tokens
        dict(net, name="block_step", kind="forward", layers=1, frames=13, rows=15, cols=22, text=226),
        # the CogVideoX-2b shape: 17550 + 226 tokens
        dict(net, name="full_step", kind="forward", frames=13, rows=30, cols=45, text=226),
        # long video: 33750 + 226 tokens
        dict(net, name="long_step", kind="forward", frames=25, rows=30, cols=45, text=226),
        # attention alone, at the block's size and at a small ragged one in a batch
        {"name": "attn_block", "kind": "attn", "batch": 1, "seq": 4516, "heads": 30, "head_dim": 64, "dtype": "bf16"},
        {"name": "attn_ragged", "kind": "attn", "batch": 2, "seq": 1000, "heads": 30, "head_dim": 64, "dtype": "bf16"},
        # the first MLP projection at the block's size
        {"name": "linear_block", "kind": "linear", "rows": 4516, "n_out": 7680, "k": 1920, "act": 1, "dtype": "bf16"},
        # bookkeeping of one step on one latent of the CogVideoX-2b shape
        {"name": "update_latent", "kind": "update", "n": 16 * 13 * 60 * 90},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "run", "run", "attn", "attn", "linear", "update"])
    if kind == "forward":
        while True:
            c = {"kind": kind, "dtype": "bf16", "layers": _log(rng, 1, 30), "frames": _log(rng, 1, 25),
                 "rows": _log(rng, 4, 30), "cols": _log(rng, 4, 45), "text": rng.choice([0, 16, 77, 226]),
                 "batch": rng.choice([1, 1, 1, 2, 4])}
            if rng.random() < 0.15:
                c.update(dtype="f32", layers=min(c["layers"], 2), frames=min(c["frames"], 3), rows=min(c["rows"], 8),
                         cols=min(c["cols"], 12), batch=1)
            if work(c)["flops"] <= 3.5e14:
                return c
    if kind == "run":
        tiny = rng.random() < 0.5
        batched = rng.random() < 0.5
        steps = rng.randint(5, 12)
        return {"kind": kind, "base": "tiny" if tiny else "reduced", "layers": 2 if tiny else _log(rng, 2, 30),
                "frames": rng.randint(1, 4), "rows": rng.randint(3, 10), "cols": rng.randint(3, 10),
                "text": rng.choice([0, 6, 16]), "dtype": "f32" if tiny else "bf16", "steps": steps,
                "warmup": rng.randint(1, 3), "window": rng.randint(2, 4), "batched": batched}
    if kind == "attn":
        if rng.random() < 0.7:
            return {"kind": kind, "batch": rng.choice([1, 1, 2]), "seq": _log(rng, 32, 17776), "heads": rng.choice([4, 16, 30]),
                    "head_dim": 64, "dtype": "bf16"}
        return {"kind": kind, "batch": rng.choice([1, 2]), "seq": _log(rng, 32, 1024), "heads": rng.choice([4, 16, 30]),
                "head_dim": rng.choice([16, 32, 64]), "dtype": "f32"}
    if kind == "linear":
        n_out, k, act = rng.choice([(5760, 1920, 0), (1920, 1920, 0), (7680, 1920, 1), (1920, 7680, 0)])
        if rng.random() < 0.15:
            return {"kind": kind, "rows": _log(rng, 8, 512), "n_out": n_out, "k": k, "act": act, "dtype": "f32"}
        return {"kind": kind, "rows": _log(rng, 8, 33976), "n_out": n_out, "k": k, "act": act, "dtype": "bf16"}
    return {"kind": kind, "n": _log(rng, 2048, 1 << 26)}


def _config(case):
    base = I.CONFIGS[{"tiny": "tiny"}.get(case.get("base"), "reduced")]
    return base.with_(layers=case["layers"], frames=case["frames"], height=2 * case["rows"], width=2 * case["cols"],
                      text_tokens=case["text"], dtype=case["dtype"])


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _weights(cfg, g):
    """The weight list of a network on the GPU: matrices in the network's type, biases fp32."""
    out, dt = [], B.torch_dtype(cfg.dtype)
    for name, shape in I.weight_shapes(cfg):
        w = torch.randn(shape, generator=g, device="cuda")
        if len(shape) == 2:
            out.append(w.mul_(shape[1] ** -0.5).to(dt))
        else:
            w.mul_(0.02)
            if name.startswith("b_mod."):                # the four gates of the layer
                w.view(12, cfg.hidden)[[2, 5, 8, 11]] += 1.0
            out.append(w)
    return out


def prepare(case, seed):
    g = _generator(seed)
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    kind = case["kind"]
    if kind in ("forward", "run"):
        cfg = _config(case)
        batch = case.get("batch", 1)
        d = B.dit_create(cfg, _weights(cfg, g))
        x = rand(batch, *cfg.latent_shape)
        ctx = rand(batch, cfg.text_tokens, cfg.hidden).to(B.torch_dtype(cfg.dtype)) if cfg.text_tokens else None
        if kind == "forward":
            ts, _, _ = B.ddim_coefficients(50)
            at = 7 + seed % 30
            d.workspace(batch)
            return {"kind": kind, "dit": d, "x": x, "ctx": ctx, "t": [int(t) for t in ts[at:at + batch]],
                    "eps": torch.empty_like(x)}
        S, m, p = case["steps"], case["warmup"], case["window"]
        ts, a, b = B.ddim_coefficients(S)
        return {"kind": kind, "dit": d, "x": x, "ctx": ctx,
                "sched": B.Schedule(ts, a, b, m, [p] * -(-(S - m) // p), batched=case["batched"])}
    dt = B.torch_dtype(case.get("dtype", "f32"))
    if kind == "attn":
        shape = (case["batch"], case["seq"], case["heads"], case["head_dim"])
        q, k, v = (rand(*shape).to(dt) for _ in range(3))
        return {"kind": kind, "q": q, "k": k, "v": v, "scale": case["head_dim"] ** -0.5, "out": torch.empty_like(q)}
    if kind == "linear":
        M, N, K = case["rows"], case["n_out"], case["k"]
        return {"kind": kind, "a": rand(M, K).to(dt), "w": (rand(N, K) * K ** -0.5).to(dt), "bias": rand(N) * 0.02,
                "act": case["act"], "out": torch.empty(M, N, dtype=dt, device="cuda")}
    n = case["n"]
    _, a, b = B.ddim_coefficients(50)
    at = 7 + seed % 30
    x, eps = rand(n), rand(n)
    return {"kind": kind, "x": x, "eps": eps, "eps_prev": eps + 0.1 * rand(n), "other": x + 0.1 * rand(n),
            "a": float(a[at]), "b": float(b[at]), "out": torch.empty_like(x)}


def run(state):
    kind = state["kind"]
    if kind == "forward":
        return B.dit_forward(state["dit"], state["x"], state["ctx"], state["t"], eps_out=state["eps"])
    if kind == "run":
        x0, sums, calls = B.sampler_run(state["dit"], state["sched"], state["x"], state["ctx"])
        return x0, sums, calls
    if kind == "attn":
        return B.attn3d(state["q"], state["k"], state["v"], state["scale"], out=state["out"])
    if kind == "linear":
        return B.dit_linear(state["a"], state["w"], state["bias"], state["act"], out=state["out"])
    x, sums = B.sampler_step(state["x"], state["eps"], state["eps_prev"], state["a"], state["b"], x_out=state["out"])
    return x, sums, B.rel_mae(state["other"], x)


def work(case):
    kind = case["kind"]
    if kind in ("forward", "run"):
        cfg = _config(case)
        es = 2 if cfg.dtype == "bf16" else 4
        batch = case.get("batch", 1)
        samples = batch if kind == "forward" else case["steps"]
        D, N, Nv, P = cfg.hidden, cfg.tokens, cfg.video_tokens, cfg.patch_dim
        weights = sum(math.prod(s) * (es if len(s) == 2 else 4) for _, s in I.weight_shapes(cfg))
        per_sample = cfg.layers * (24 * N * D * D + 4 * N * N * D) + 4 * Nv * P * D
        flops = samples * per_sample + 2 * cfg.layers * 12 * D * cfg.time_embed_dim * samples
        return {"bytes": weights + batch * (8 * cfg.latent_elems + es * cfg.text_tokens * D), "flops": flops}
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "attn":
        rows = case["batch"] * case["seq"] * case["heads"]
        return {"bytes": 4 * rows * case["head_dim"] * es, "flops": 4 * rows * case["seq"] * case["head_dim"]}
    if kind == "linear":
        M, N, K = case["rows"], case["n_out"], case["k"]
        return {"bytes": es * (M * K + N * K + M * N) + 4 * N, "flops": 2 * M * N * K}
    return {"bytes": 4 * 5 * case["n"], "flops": 12 * case["n"]}


def tolerance(case):
    # about four times what was measured: fp32 calls against float64 sums 7e-7 (attention) to 1.6e-6 (projections); the
    # bf16 network against itself in fp32 3.4e-3 (1.2e-2 at most) and against other softmax and tile paths 4e-3 (1.7e-2);
    # bf16 attention and projections against float64 2.3e-3 (1.2e-2); the update and its sums against float64 5e-8
    if case["kind"] == "update":
        return {"rel": 1e-6}
    if case.get("dtype") == "f32":
        return {"rel": 1e-5}
    if case["kind"] in ("forward", "run"):
        return {"rel": 1.5e-2, "max": 7e-2}
    return {"rel": 1e-2, "max": 5e-2}


# ---- the same results in 64 bits, in plain torch

def _exact_ddim(steps):
    abar = torch.cumprod(1.0 - torch.linspace(1e-4, 2e-2, 1000, dtype=torch.float64), 0)
    ts = [(steps - 1 - i) * (1000 // steps) for i in range(steps)]
    prev = [abar[t].item() for t in ts[1:]] + [1.0]
    a = [math.sqrt(p / abar[t].item()) for t, p in zip(ts, prev)]
    b = [math.sqrt(1.0 - p) - f * math.sqrt(1.0 - abar[t].item()) for t, p, f in zip(ts, prev, a)]
    return ts, a, b


def _exact_attention(q, k, v, scale):
    """[N, H, d] each; a head at a time, in blocks of query rows."""
    out = torch.empty_like(q)
    for h in range(q.shape[1]):
        kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
        for r in range(0, q.shape[0], 4096):
            out[r:r + 4096, h] = torch.softmax(q[r:r + 4096, h].contiguous() @ kt * scale, -1) @ vh
    return out


def _exact_forward(cfg, weights, x, ctx, t):
    """One sample: x [C, F, H, W], ctx [L, D] or None, t an integer."""
    wide = lambda w: w.to(torch.float64)
    silu = lambda u: u * torch.sigmoid(u)
    ln = lambda u: torch.nn.functional.layer_norm(u, (u.shape[-1],), eps=cfg.ln_eps)
    D, L, ps = cfg.hidden, cfg.text_tokens, cfg.patch
    C, F, H, W = cfg.latent_shape
    Hp, Wp, d = H // ps, W // ps, cfg.head_dim
    it = iter(weights)
    lin = lambda u: u @ wide(next(it)).t() + wide(next(it))
    patches = x.reshape(C, F, Hp, ps, Wp, ps).permute(1, 2, 4, 0, 3, 5).reshape(F * Hp * Wp, -1)
    X = lin(patches)
    if L:
        X = torch.cat([wide(ctx), X])
    w = torch.exp(-torch.arange(D // 2, dtype=torch.float64, device=x.device) / (D // 2) * math.log(10000.0))
    c = silu(lin(silu(lin(torch.cat([torch.cos(t * w), torch.sin(t * w)])))))
    grid = torch.meshgrid(*(torch.arange(n, dtype=torch.float64, device=x.device) for n in (F, Hp, Wp)), indexing="ij")
    ang = [p.reshape(-1, 1) * cfg.rope_theta ** (-2.0 * torch.arange(n // 2, dtype=torch.float64, device=x.device) / n)
           for p, n in zip(grid, (d // 4, 3 * d // 8, 3 * d // 8))]
    rot = torch.polar(torch.ones((), dtype=torch.float64, device=x.device), torch.cat(ang, 1))[:, None, :]

    def turned(u):
        v = torch.view_as_complex(u[L:].reshape(-1, cfg.heads, d // 2, 2).contiguous()) * rot
        return torch.cat([u[:L], torch.view_as_real(v).reshape(-1, cfg.heads, d)])

    for _ in range(cfg.layers):
        mod = lin(c).view(2, 6, D)                      # video, text
        m = [torch.cat([mod[1, i].expand(L, D), mod[0, i].expand(X.shape[0] - L, D)]) for i in range(6)]
        q, k, v = (u.reshape(-1, cfg.heads, d) for u in lin(ln(X) * (1 + m[1]) + m[0]).split(D, 1))
        X = X + m[2] * lin(_exact_attention(turned(q), turned(k), v, d ** -0.5).reshape(-1, D))
        u = torch.nn.functional.gelu(lin(ln(X) * (1 + m[4]) + m[3]), approximate="tanh")
        X = X + m[5] * lin(u)
    shift, scale = lin(c).split(D)
    out = lin(ln(X[L:]) * (1 + scale) + shift)
    return out.reshape(F, Hp, Wp, C, ps, ps).permute(3, 0, 1, 4, 2, 5).reshape(C, F, H, W)


def _exact_run(case, cfg, weights, x, ctx):
    ts, a, b = _exact_ddim(case["steps"])
    predict = lambda y, i: _exact_forward(cfg, weights, y, ctx, ts[i])
    step = lambda y, e, i: y + ((a[i] - 1.0) * y + b[i] * e)
    sums, last, i, calls = [], None, 0, 0
    cache = [None] * case["window"]

    def take(y, e, i):
        new = step(y, e, i)
        zero = torch.zeros((), dtype=torch.float64, device=y.device)
        sums.append(torch.stack([(new - y).abs().sum(), new.abs().sum(), (e - last).abs().sum() if last is not None else zero,
                                 e.abs().sum()]))
        return new

    while i < min(case["warmup"], case["steps"]):
        e = predict(x, i)
        x, last, cache, calls, i = take(x, e, i), e, [e] * case["window"], calls + 1, i + 1
    while i < case["steps"]:
        n = min(case["window"], case["steps"] - i)
        eps = []
        for r in range(n):                              # rank r's sample: advanced r times with what it predicted last
            y = x
            for j in range(r):
                y = step(y, cache[r], i + j)
            eps.append(predict(y, i + r))
        for r in range(n):
            x, last, cache[r] = take(x, eps[r], i + r), eps[r], eps[r]
        i, calls = i + n, calls + (1 if case["batched"] else n)
    return x, torch.stack(sums), calls


def exact(case, seed):
    """What `run` returns, in 64 bits; None where that would take too long."""
    kind = case["kind"]
    if work(case)["flops"] > 5e13:
        return None
    s = prepare(case, seed)
    wide = lambda u: u.to(torch.float64)
    if kind in ("forward", "run"):
        cfg, weights, ctx = _config(case), s["dit"].weights, s["ctx"]
        if kind == "forward":
            return torch.stack([_exact_forward(cfg, weights, wide(s["x"][i]), None if ctx is None else ctx[i], s["t"][i])
                                for i in range(case["batch"])])
        x, sums, calls = _exact_run(case, cfg, weights, wide(s["x"][0]), None if ctx is None else ctx[0])
        return x[None], sums, calls
    if kind == "attn":
        return torch.stack([_exact_attention(wide(s["q"][i]), wide(s["k"][i]), wide(s["v"][i]), s["scale"])
                            for i in range(case["batch"])])
    if kind == "linear":
        out = wide(s["a"]) @ wide(s["w"]).t() + wide(s["bias"])
        return torch.nn.functional.gelu(out, approximate="tanh") if case["act"] else out
    x, eps = wide(s["x"]), wide(s["eps"])
    delta = (s["a"] - 1.0) * x + s["b"] * eps
    new, other = x + delta, wide(s["other"])
    sums = torch.stack([delta.abs().sum(), new.abs().sum(), (eps - wide(s["eps_prev"])).abs().sum(), eps.abs().sum()])
    mae = torch.stack([(other - new).abs().sum(), other.abs().sum()])
    return new, sums, torch.cat([mae, mae[:1] / mae[1:]])

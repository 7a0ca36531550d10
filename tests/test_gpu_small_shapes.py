"""Kernels for few tokens and for fp32 operands at the sizes where they can go wrong: edges of 64 x 64 tiles, K pieces of
unequal length, pieces added by the following LayerNorm, ragged keys, more predictor steps than one conditioning chunk."""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import parastep_oracle as O
from paper_2505_14741_amd import binding as B
from paper_2505_14741_amd import inputs as I

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rel(ref, out):
    return float(np.linalg.norm(out.astype(np.float64) - ref) / np.linalg.norm(ref))


# bounds: fp32 sums of K products, error at most about sqrt(K) * 2^-24 of the result's norm (K = 7680: 5e-6); bf16 results
# are rounded once, 2^-9 at most
@pytest.mark.parametrize("M", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("Nn,K", [(64, 64), (68, 320), (196, 1984), (1920, 7680), (4, 96)])
@pytest.mark.parametrize("act", [0, 1])
def test_linear_few_rows_split_and_whole(M, Nn, K, act):
    print(f"dit_linear M={M} N={Nn} K={K} act={act}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M * 7 + Nn)
    for td, bound in ((torch.float32, 5e-6), (torch.bfloat16, 2.0 ** -9)):
        a = torch.randn(M, K, generator=g, device=DEV).to(td)
        w = (torch.randn(Nn, K, generator=g, device=DEV) / math.sqrt(K)).to(td)
        bias = torch.randn(Nn, generator=g, device=DEV)
        ref = a.double() @ w.double().t() + bias.double()
        if act:
            ref = torch.nn.functional.gelu(ref, approximate="tanh")
        ref = ref.cpu().numpy()
        for kw in ({}, {"use_workspace": False}, {"kernel_path": 4}):     # in K pieces, and whole both ways
            assert rel(ref, B.dit_linear(a, w, bias, act, **kw).double().cpu().numpy()) <= bound, (td, kw)


@pytest.mark.parametrize("N", [768, 769, 960, 961, 1088, 1152, 1153, 1280, 1281, 1344, 1408])
def test_linear_on_both_sides_of_the_tile_limit(N):
    """1920 columns are 30 column tiles of 64: 21 and 22 row tiles are 630 and 660, around the limit of 640 for K = 1920.  K =
    7680 is cut in 4 pieces up to 768 rows and from 961 to 1152, in 3 between and up to 1280, and not beyond; the tiles of the
    other kernel, forced, add the same pieces.  One rounding of the result to bf16."""
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    for K in (1920, 7680):
        a = torch.randn(N, K, generator=g, device=DEV).bfloat16()
        w = (torch.randn(1920, K, generator=g, device=DEV) / math.sqrt(K)).bfloat16()
        bias = torch.randn(1920, generator=g, device=DEV)
        ref = (a.double() @ w.double().t() + bias.double()).cpu().numpy()
        out = B.dit_linear(a, w, bias, 0)
        assert rel(ref, out.double().cpu().numpy()) <= 2.0 ** -9
        assert rel(ref, B.dit_linear(a, w, bias, 0, use_workspace=False).double().cpu().numpy()) <= 2.0 ** -9
        if N <= 1280 or K == 1920:                       # (above, 128 x 128 tiles have a last round of their own to cut)
            assert torch.equal(out, B.dit_linear(a, w, bias, 0, kernel_path=0x200))


# rows, columns, K that between them take every tile of the few-token kernel
TILE_SIZES = [(300, 1908, 1920), (700, 1908, 1920), (1290, 1908, 1920), (2500, 1908, 1920), (3300, 1908, 7680), (4500, 1908, 7680)]


@pytest.mark.parametrize("M,Nn,K", TILE_SIZES)
def test_every_tile_of_the_few_token_kernel_at_ragged_edges(M, Nn, K):
    """Rows and columns that end inside a tile, more row tiles than a band of 8; whole sums, so a forced tile of the other
    kernel gives the same bits.  One rounding of the result to bf16."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    a = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    w = (torch.randn(Nn, K, generator=g, device=DEV) / math.sqrt(K)).bfloat16()
    bias = torch.randn(Nn, generator=g, device=DEV)
    out = B.dit_linear(a, w, bias, 0)
    ref = a.double() @ w.double().t() + bias.double()
    assert rel(ref.cpu().numpy(), out.double().cpu().numpy()) <= 2.0 ** -9
    assert torch.equal(out, B.dit_linear(a, w, bias, 0, kernel_path=0x204))


@pytest.mark.parametrize("M,Nn,K", [(300, 260, 64), (300, 260, 128), (300, 260, 192), (300, 260, 4032), (300, 260, 4096),
                                    (3300, 4100, 4032), (3300, 4100, 4096), (4200, 4100, 4160)])
def test_rings_of_the_wide_tiles(M, Nn, K):
    """Two and three stages of either operand: K of one to three stages, short and long K on both sides of the line, one round of
    workgroups and more; whole sums, so every ring gives the bits of the 128 x 128 tile.  One rounding of the result to bf16."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    a = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    w = (torch.randn(Nn, K, generator=g, device=DEV) / math.sqrt(K)).bfloat16()
    bias = torch.randn(Nn, generator=g, device=DEV)
    out = B.dit_linear(a, w, bias, 0, kernel_path=0x204)
    ref = a[-300:].double() @ w.double().t() + bias.double()
    assert rel(ref.cpu().numpy(), out[-300:].double().cpu().numpy()) <= 2.0 ** -9
    for variant in (1, 3):
        assert torch.equal(out, B.dit_linear(a, w, bias, 0, kernel_path=variant << 8 | 4)), variant


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 384])
@pytest.mark.parametrize("M,Nn", [(40, 196), (300, 3900), (600, 3900)])
def test_fewer_stages_than_the_ring_and_a_few_more(M, Nn, K):
    """The stages after the steady state are written out: K of one to six stages on 64 x 64, 128 x 64 and 128 x 128 tiles of the
    few-token kernel and on every tile of the other (same bits), fp32 on its own.  One rounding of the result to bf16; fp32 sums
    as above."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    for td, bound in ((torch.float32, 5e-6), (torch.bfloat16, 2.0 ** -9)):
        a = torch.randn(M, K, generator=g, device=DEV).to(td)
        w = (torch.randn(Nn, K, generator=g, device=DEV) / math.sqrt(K)).to(td)
        bias = torch.randn(Nn, generator=g, device=DEV)
        out = B.dit_linear(a, w, bias, 0)
        assert rel((a.double() @ w.double().t() + bias.double()).cpu().numpy(), out.double().cpu().numpy()) <= bound
        for variant in (1, 2, 3, 4) if td == torch.bfloat16 and M > 40 else ():      # (few rows: in K pieces)
            assert torch.equal(out, B.dit_linear(a, w, bias, 0, kernel_path=variant << 8)), variant


@pytest.mark.parametrize("M", [3, 70, 700])
def test_linear_of_operand_rows_longer_than_8_mb(M):
    """The rows of one 64 x 64 tile are half a GB apart from first to last; edges inside a tile and past it.  fp32 sums as above."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    for td, K in ((torch.float32, (1 << 21) + 32), (torch.bfloat16, (1 << 22) + 64)):
        print(f"dit_linear M={M} N=68 K={K}", flush=True)
        a = torch.randn(M, K, generator=g, device=DEV, dtype=td)
        w = torch.randn(68, K, generator=g, device=DEV, dtype=td).mul_(K ** -0.5)
        bias = torch.randn(68, generator=g, device=DEV)
        ref = bias.double().expand(M, 68).clone()
        for k in range(0, K, 1 << 18):
            ref += a[:, k:k + (1 << 18)].double() @ w[:, k:k + (1 << 18)].double().t()
        bound = 5e-6 * (K / 7680) ** 0.5 + (2.0 ** -9 if td == torch.bfloat16 else 0)
        for kw in ({}, {"use_workspace": False}, {"kernel_path": 0x200}):
            assert rel(ref.cpu().numpy(), B.dit_linear(a, w, bias, 0, **kw).double().cpu().numpy()) <= bound, (td, kw)


@pytest.mark.parametrize("N", [1, 15, 16, 17, 63, 64, 65, 200])
@pytest.mark.parametrize("d", [16, 32, 64])
def test_attention_fp32_math_ragged(N, d):
    """fp32, and bf16 at the head dims that run with fp32 math (one rounding of the result); logits of order 10 in one head."""
    g = torch.Generator(device=DEV)
    g.manual_seed(N + d)
    for td, bound in ((torch.float32, 2e-6), (torch.bfloat16, 2.0 ** -9)):
        if td == torch.bfloat16 and d == 64:
            continue
        q, k, v = (torch.randn(2, N, 3, d, generator=g, device=DEV).to(td) for _ in range(3))
        q[:, :, 1] *= 4.0
        out = B.attn3d(q, k, v, d ** -0.5)
        s = torch.einsum("bqhd,bkhd->bhqk", q.double().cpu(), k.double().cpu()) * d ** -0.5
        ref = torch.einsum("bhqk,bkhd->bqhd", torch.softmax(s, -1), v.double().cpu()).numpy()
        assert rel(ref, out.double().cpu().numpy()) <= bound


@pytest.mark.parametrize("N", [512, 513, 1024, 4096])
def test_attention_bf16_with_few_items(N):
    """4 heads, 8 with both samples: workgroups of 128 queries, whatever the number of keys; the batch changes no bit."""
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    q, k, v = (torch.randn(2, N, 4, 64, generator=g, device=DEV).bfloat16() for _ in range(3))
    out = B.attn3d(q, k, v, 0.125)
    assert torch.equal(B.attn3d(q[1:], k[1:], v[1:], 0.125)[0], out[1])
    rows = torch.tensor([0, 1, N // 2, N - 1])
    for b in range(2):
        for h in range(4):
            kd, vd = k[b, :, h].double().cpu(), v[b, :, h].double().cpu()
            ref = (torch.softmax(q[b, rows, h].double().cpu() @ kd.t() * 0.125, -1) @ vd).numpy()
            # probabilities and result in bf16: two roundings of 2^-9
            assert rel(ref, out[b, rows, h].double().cpu().numpy()) <= 2 * 2.0 ** -9


@pytest.mark.parametrize("N", [31, 129, 300, 1000])
def test_attention_queries_that_overflow_are_redone_alone(N):
    """Logits far beyond what fits without a softmax reference, in some queries of one head: the workgroups of 128 queries
    redo theirs on the spot, those of 256 (16 samples of 1000 keys) leave them to a second launch; the other queries of the
    workgroup keep their values, and the batch changes no bit."""
    H = 16
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    q, k, v = (torch.randn(16, N, H, 64, generator=g, device=DEV).bfloat16() for _ in range(3))
    plain = B.attn3d(q, k, v, 0.125).clone()
    big = [r for r in (5, 30, 128, 299, 700) if r < N]
    q[3, big, 2] *= 200.0
    q[3, big[:1], 2] = -q[3, big[:1], 2]
    out = B.attn3d(q, k, v, 0.125)
    for b in (2, 3, 15):
        assert torch.equal(B.attn3d(q[b:b + 1], k[b:b + 1], v[b:b + 1], 0.125)[0], out[b]), b
    ref = torch.softmax(q[3, :, 2].double().cpu() @ k[3, :, 2].double().cpu().t() * 0.125, -1) @ v[3, :, 2].double().cpu()
    assert rel(ref.numpy(), out[3, :, 2].double().cpu().numpy()) <= 2 * 2.0 ** -9
    near = {r // 32 for r in big}                        # the groups of 32 queries that are redone
    same = [r for r in range(N) if r // 32 not in near]
    assert torch.equal(out[3, same, 2], plain[3, same, 2])
    assert torch.equal(out[:3], plain[:3]) and torch.equal(out[4:], plain[4:])
    v[3, :, 2] = float("nan")                            # a head that stays NaN, and no other
    assert torch.isnan(B.attn3d(q, k, v, 0.125)[3, :, 2]).all()


@pytest.mark.parametrize("text", [0, 6, 70])
@pytest.mark.parametrize("frames,rows,cols", [(1, 3, 3), (2, 8, 8), (3, 5, 7)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_forward_few_tokens(dtype, frames, rows, cols, text):
    """Text rows and video rows in one tile, tiles of text only, token counts off the tile; both types against the oracle."""
    base = I.CONFIGS["tiny_text"] if dtype == "f32" else I.CONFIGS["reduced"].with_(layers=2)
    cfg = base.with_(frames=frames, height=2 * rows, width=2 * cols, text_tokens=text)
    print(f"forward {dtype} tokens {cfg.tokens} text {text}", flush=True)
    W = I.make_weights(cfg, 1001, "unit")
    d = B.dit_create(cfg, B.weights_to_device(cfg, W, DEV))
    x, ctx = I.make_latent(cfg, 2), I.make_context(cfg, 2) if text else None
    ctxd = torch.from_numpy(ctx).to(DEV).to(B.torch_dtype(dtype)) if text else None
    xd = torch.from_numpy(x).to(DEV)
    eps = B.dit_forward(d, xd, ctxd, [900, 20])
    ref = O.dit_forward(cfg, dict(W), x, ctx, [900, 20])
    for b in range(2):
        assert O.rel_mae(ref[b], eps[b].cpu().numpy())[2] <= (1e-4 if dtype == "f32" else 2e-2)
        one = B.dit_forward(d, xd[b:b + 1].contiguous(), None if ctxd is None else ctxd[b:b + 1].contiguous(), [[900, 20][b]])
        assert torch.equal(one[0], eps[b])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("channels,patch", [(1, 2), (4, 2), (3, 4), (16, 2), (20, 2), (4, 1)])
def test_patch_vectors_of_any_length(dtype, channels, patch):
    """bf16 weights: up to 64 values per patch as three bf16 parts of every pixel, longer ones (80) and fp32 weights in fp32
    products.  Pixels from 2^-12 to 2^12; 77 columns of patches and 70 text rows end inside a tile.  Output projections of
    zero leave the embedding to the final layer, whose rounding to bf16 is one in 2^9 per value."""
    cfg = I.CONFIGS["reduced"].with_(layers=1, frames=1, height=4 * patch, width=77 * patch, in_channels=channels, patch=patch,
                                     text_tokens=70, dtype=dtype)
    W = [(n, w * 0 if n.split(".")[0] in ("W_o", "b_o", "W_2", "b_2") else w) for n, w in I.make_weights(cfg, 1001, "unit")]
    assert sum(float(np.abs(w).max()) == 0 for _, w in W) == 4
    d = B.dit_create(cfg, B.weights_to_device(cfg, W, DEV))
    rng = np.random.default_rng(channels * patch)
    x = (I.make_latent(cfg, 2) * 2.0 ** rng.integers(-12, 13, size=(2,) + tuple(cfg.latent_shape))).astype(np.float32)
    ctx = I.make_context(cfg, 2)
    eps = B.dit_forward(d, torch.from_numpy(x).to(DEV), torch.from_numpy(ctx).to(DEV).to(B.torch_dtype(dtype)), [900, 20])
    ref = O.dit_forward(cfg, dict(W), x, ctx, [900, 20])
    assert rel(ref, eps.cpu().numpy()) <= (1e-5 if dtype == "f32" else 2.0 ** -8)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("channels,patch", [(1, 2), (4, 2), (3, 4), (16, 2), (20, 2)])
def test_embedding_loses_nothing_of_a_pixel(dtype, channels, patch):
    """The residual stream, at the head of the workspace, holds the embedding itself where the layer's output projections are
    zero.  One pixel per patch: its product with a weight, rounded to fp32 (one step of the last place, 2^-23, for a sum that is
    rounded otherwise); a pixel without its last 8 bits would be off by up to 2^-15.  All pixels: fp32 sums of at most 3 * 80
    terms, sqrt(240) * 2^-24 of the result's norm; without the last 8 bits of the pixels it would be 2^-17.  Text rows exactly."""
    cfg = I.CONFIGS["reduced"].with_(layers=1, frames=1, height=4 * patch, width=77 * patch, in_channels=channels, patch=patch,
                                     text_tokens=70, dtype=dtype)
    td, P = B.torch_dtype(dtype), cfg.patch_dim
    g = torch.Generator(device=DEV)
    g.manual_seed(channels)
    rand = lambda *shape: torch.randn(shape, generator=g, device=DEV)
    named = [(n, rand(*shape)) for n, shape in I.weight_shapes(cfg)]
    named = [(n, w * 0 if n.split(".")[0] in ("W_o", "b_o", "W_2", "b_2", "b_pe") else w) for n, w in named]
    assert sum(not w.any() for _, w in named) == 5
    weights = [(w * w.shape[1] ** -0.5).to(td) if w.dim() == 2 else w for _, w in named]
    W_pe = dict(zip([n for n, _ in named], weights))["W_pe"].double()
    d = B.dit_create(cfg, weights)
    ctx = rand(2, 70, cfg.hidden).to(td)
    patches = rand(2, cfg.video_tokens, P) * 2.0 ** torch.randint(-6, 7, (2, cfg.video_tokens, P), generator=g, device=DEV)
    one = torch.zeros_like(patches)
    token = torch.arange(cfg.video_tokens, device=DEV)
    one[:, token, token % P] = patches[:, token, token % P]
    for p, whole in ((one, False), (patches, True)):
        Hp, Wp = cfg.height // patch, cfg.width // patch
        x = p.view(2, 1, Hp, Wp, channels, patch, patch).permute(0, 4, 1, 2, 5, 3, 6).reshape(2, *cfg.latent_shape).contiguous()
        B.dit_forward(d, x, ctx, [900, 20])
        X = d.workspace(2)[:8 * cfg.tokens * cfg.hidden].view(torch.float32).view(2, cfg.tokens, cfg.hidden)
        assert torch.equal(X[:, :70], ctx.float())
        ref = torch.matmul(p.double().view(-1, P), W_pe.t()).view(2, cfg.video_tokens, cfg.hidden)
        err = (X[:, 70:].double() - ref).abs()
        if whole:
            assert err.norm() <= 240 ** 0.5 * 2.0 ** -24 * ref.norm()
        else:
            assert (err <= 2.0 ** -23 * ref.abs()).all()


@pytest.mark.parametrize("mode,batched,S,m,cyc", [(0, False, 37, 3, [4] * 9), (1, False, 37, 1, [3] * 12), (0, True, 37, 2, [7] * 5)])
def test_run_longer_than_one_conditioning_chunk(mode, batched, S, m, cyc):
    """More predictor calls than the 16 whose modulation is computed together: step by step (one at a time) equals the whole
    run bit for bit."""
    cfg = I.CONFIGS["tiny_text"]
    d = B.dit_create(cfg, B.weights_to_device(cfg, I.make_weights(cfg, 1001, "unit"), DEV))
    x_T = torch.from_numpy(I.make_latent(cfg, 1)).to(DEV)
    ctx = torch.from_numpy(I.make_context(cfg, 1)).to(DEV)
    ts, a, b = B.ddim_coefficients(S)
    sched = B.Schedule(ts, a, b, m, cyc, batched=batched, mode=mode)
    x0, sums, _ = B.sampler_run(d, sched, x_T, ctx)
    ws, state, out, sums2 = B.sampler_workspace(d, sched, DEV), B.SamplerState(), torch.empty_like(x_T), torch.zeros_like(sums)
    stops = list(range(1, S + 1)) if not batched else list(range(1, m + 1)) + [min(S, m + 7 * (i + 1)) for i in range(5)]
    for stop in stops:
        B.sampler_run_steps(d, sched, state, stop, x_T, ctx, ws, out, sums2)
    assert torch.equal(out, x0) and torch.equal(sums2, sums)


def graph_nodes(call):
    """How many kernels a call enqueues: the nodes of the graph it is captured into."""
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = ctypes.c_size_t()
    hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64.so" in l)      # the runtime that is in use
    assert ctypes.CDLL(hip).hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def test_modulation_off_the_matrix_path_is_one_launch_per_32_layers():
    """40 layers: the matrix kernel takes 41 matrices in 2 launches; time_embed_dim 72 takes 32 + 8 + the final one."""
    def nodes(Dt):
        cfg = I.CONFIGS["tiny_text"].with_(time_embed_dim=Dt, layers=40)
        d = B.dit_create(cfg, B.weights_to_device(cfg, I.make_weights(cfg, 1001, "unit"), DEV))
        x, ctx = torch.from_numpy(I.make_latent(cfg, 1)).to(DEV), torch.from_numpy(I.make_context(cfg, 1)).to(DEV)
        return graph_nodes(lambda: B.dit_forward(d, x, ctx, [500]))
    assert nodes(72) == nodes(64) + 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_modulation_of_many_layers_equals_that_of_one(dtype):
    """Beyond 200000 rows of modulation matrices (9 layers of width 1920) a wave takes 32 rows at a time instead of 16, with
    the same values: of 9 layers all but one add nothing, wherever that one stands the network equals it alone bit for bit."""
    one = I.CONFIGS["reduced"].with_(layers=1, frames=1, height=2, width=6, text_tokens=8, dtype=dtype)
    nine = one.with_(layers=9)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    td = B.torch_dtype(dtype)
    rand = [torch.randn(shape, generator=g, device=DEV).mul_(shape[1] ** -0.5).to(td) if len(shape) == 2
            else torch.randn(shape, generator=g, device=DEV) for _, shape in I.weight_shapes(one)]
    head, layer, tail = rand[:6], rand[6:16], rand[16:]
    # order of a layer: W_mod b_mod W_qkv b_qkv W_o b_o W_1 b_1 W_2 b_2; without output projections it adds nothing
    idle = [torch.zeros_like(t) if i in (4, 5, 8, 9) else t for i, t in enumerate(layer)]
    x = torch.randn(3, *one.latent_shape, generator=g, device=DEV)
    ctx = torch.randn(3, 8, one.hidden, generator=g, device=DEV).to(td)
    t = [900, 400, 20]
    ref = B.dit_forward(B.dit_create(one, rand), x, ctx, t).clone()
    assert torch.isfinite(ref).all()
    for at in (0, 4, 8):
        w = head + [t for l in range(9) for t in (layer if l == at else idle)] + tail
        assert torch.equal(B.dit_forward(B.dit_create(nine, w), x, ctx, t), ref), at


@pytest.mark.parametrize("Dt", [64, 72, 1024])
def test_modulation_widths_on_and_off_the_matrix_path(Dt):
    """time_embed_dim a multiple of 64 up to 1000 takes the matrix kernel, others vector products."""
    cfg = I.CONFIGS["tiny_text"].with_(time_embed_dim=Dt)
    W = I.make_weights(cfg, 1001, "unit")
    d = B.dit_create(cfg, B.weights_to_device(cfg, W, DEV))
    x, ctx = I.make_latent(cfg, 3), I.make_context(cfg, 3)
    eps = B.dit_forward(d, torch.from_numpy(x).to(DEV), torch.from_numpy(ctx).to(DEV), [900, 500, 20])
    ref = O.dit_forward(cfg, dict(W), x, ctx, [900, 500, 20])
    assert O.rel_mae(ref, eps.cpu().numpy())[2] <= 1e-4


@pytest.mark.parametrize("n", [1, 5, 4095, 4096, 4097])
def test_update_and_rel_mae_on_one_and_two_workgroups(n):
    """Up to 4096 elements one workgroup writes the sums itself; a thread adds at most 16 values in fp32, the rest is double."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    x, e, ep = (torch.randn(n, generator=g, device=DEV) for _ in range(3))
    out, sums = B.sampler_step(x, e, ep, 1.01, -0.05)
    xd, ed = x.double(), e.double()
    dl = 0.01 * xd - 0.05 * ed
    ref = torch.stack([dl.abs().sum(), (xd + dl).abs().sum(), (ed - ep.double()).abs().sum(), ed.abs().sum()])
    assert torch.allclose(sums.double(), ref, rtol=16 * 2.0 ** -23, atol=0)
    r = B.rel_mae(x, e).double()
    num, den = (xd - ed).abs().sum(), xd.abs().sum()
    assert torch.allclose(r, torch.stack([num, den, num / den]), rtol=16 * 2.0 ** -23, atol=0)
    assert torch.isnan(B.rel_mae(torch.zeros(n, device=DEV), torch.zeros(n, device=DEV))[2])


BATCH_GRIDS = [(1, 3), (6, 8), (12, 20), (18, 28), (24, 32), (28, 39), (28, 44), (30, 43), (36, 43), (40, 51), (48, 54)]


@pytest.mark.parametrize("dtype,rows,cols", [("bf16", *g) for g in BATCH_GRIDS] + [("f32", *g) for g in BATCH_GRIDS[:5]])
def test_forward_of_a_batch_equals_single_calls_whatever_kernels_the_batch_takes(dtype, rows, cols):
    """One block of width 1920.  What runs a projection or a LayerNorm depends on the rows of the whole batch (K pieces in
    workgroups of their own or in registers, 64- or 128-wide tiles, a row per workgroup or per wave), its values do not:
    samples of 11 to 2600 tokens (fp32, one kernel
    for every size: to 776), batches of 1, 2, 5 and 16, bit for bit."""
    cfg = I.CONFIGS["reduced"].with_(layers=1, frames=1, height=2 * rows, width=2 * cols, text_tokens=8, dtype=dtype)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * cols)
    td = B.torch_dtype(dtype)
    w = []
    for name, shape in I.weight_shapes(cfg):
        t = torch.randn(shape, generator=g, device=DEV)
        w.append((t * shape[1] ** -0.5).to(td) if len(shape) == 2 else t)
    d = B.dit_create(cfg, w)
    x = torch.randn(16, *cfg.latent_shape, generator=g, device=DEV)
    ctx = torch.randn(16, cfg.text_tokens, cfg.hidden, generator=g, device=DEV).to(td)
    t = [60 * b + 7 for b in range(16)]
    one = [B.dit_forward(d, x[b:b + 1].contiguous(), ctx[b:b + 1].contiguous(), [t[b]])[0].clone() for b in range(16)]
    assert torch.isfinite(one[0]).all()
    for n in (2, 5, 16):
        print(f"forward {dtype} {cfg.tokens} tokens, batch {n}", flush=True)
        out = B.dit_forward(d, x[:n].contiguous(), ctx[:n].contiguous(), t[:n])
        for b in range(n):
            assert torch.equal(out[b], one[b]), (n, b)


@pytest.mark.parametrize("hidden,heads,channels,patch", [(32, 1, 4, 2), (32, 2, 16, 1), (64, 2, 12, 2), (64, 4, 16, 2)])
@pytest.mark.parametrize("frames,rows,cols,text", [(1, 1, 4, 0), (1, 3, 5, 0), (1, 4, 4, 16), (2, 7, 9, 17), (16, 8, 8, 0)])
@pytest.mark.parametrize("layers", [1, 3])
def test_narrow_network_in_one_launch_per_layer(hidden, heads, channels, patch, frames, rows, cols, text, layers):
    """Row blocks of 16 tokens that end inside, at and before the last token, text and video rows in one block, keys past a
    tile of 64, 1 to 4 blocks of patch values, up to the 1024 tokens it serves: against the oracle, and the batch changes no
    bit."""
    cfg = I.CONFIGS["tiny_text"].with_(layers=layers, hidden=hidden, heads=heads, head_dim=hidden // heads, frames=frames,
                                       height=rows * patch, width=cols * patch, in_channels=channels, patch=patch, text_tokens=text)
    W = I.make_weights(cfg, 1001, "unit")
    d = B.dit_create(cfg, B.weights_to_device(cfg, W, DEV))
    x, ctx = I.make_latent(cfg, 2), I.make_context(cfg, 2) if text else None
    xd, cd = torch.from_numpy(x).to(DEV), torch.from_numpy(ctx).to(DEV) if text else None
    eps = B.dit_forward(d, xd, cd, [900, 20])
    ref = O.dit_forward(cfg, dict(W), x, ctx, [900, 20])
    for b in range(2):
        assert O.rel_mae(ref[b], eps[b].cpu().numpy())[2] <= 1e-5          # fp32 sums of up to 256 and 1024 terms, 3 layers
        one = B.dit_forward(d, xd[b:b + 1].contiguous(), None if cd is None else cd[b:b + 1].contiguous(), [[900, 20][b]])
        assert torch.equal(one[0], eps[b])
    assert graph_nodes(lambda: B.dit_forward(d, xd, cd, [900, 20])) == 4 + 1 + layers


@pytest.mark.parametrize("mode", [1, 2])
def test_profile_of_a_narrow_network_and_of_one_that_is_not(mode):
    """A narrow network's launches -- tables, two layers of the time MLP, modulation, embedding, one per layer -- all count as
    "everything else", on the generic kernels and in a wider network a layer's operations count one by one; profiling changes
    no value."""
    narrow = I.CONFIGS["tiny_text"].with_(layers=3)
    for cfg, path, one_launch in ((narrow, 0, True), (narrow, 1, False), (narrow.with_(hidden=128, heads=8), 0, False)):
        d = B.dit_create(cfg, B.weights_to_device(cfg, I.make_weights(cfg, 1001, "unit"), DEV))
        B.dit_set_kernel_path(d, path)
        x, ctx = torch.from_numpy(I.make_latent(cfg, 1)).to(DEV), torch.from_numpy(I.make_context(cfg, 1)).to(DEV)
        plain = B.dit_forward(d, x, ctx, [500]).clone()
        B.dit_profile_enable(d, mode)
        assert torch.equal(B.dit_forward(d, x, ctx, [500]), plain)
        prof = B.dit_profile_read(d)
        B.dit_profile_enable(d, 0)
        for name, (ms, count) in prof.items():
            layers = 0 if one_launch else 3
            want = layers if name == "attention" else 0 if mode == 2 else None if name in ("ln_modulate", "other") else layers
            assert (ms > 0) == (count > 0), name
            assert want is None or count == want, (name, count)
        if mode == 1:
            assert prof["ln_modulate"][1] == 0 if one_launch else prof["ln_modulate"][1] >= 6
            assert prof["other"][1] == 4 + 1 + 3 if one_launch else prof["other"][1] > 0


@pytest.mark.parametrize("rows", [5, 64])
def test_fp32_gelu_over_its_range(rows):
    """The fp32 GELU epilogue alone (zero product, the value in the bias): both tails, the cut where its quotient is no longer
    refined, zeros, infinity and NaN, against float64.  A result of a few operations of one rounding each: 8 units in the last
    place of the larger of result and 1/8 of the argument (the exponent's rounding, up to |t| * 2^-24 of a factor below 1)."""
    v = np.concatenate([np.linspace(-14, 14, 449), [-1e4, -3e18, 0.0, -0.0, 1e-30, -1e-30, 1e4, 3e18, np.inf, np.nan], np.linspace(-7, -4, 53)])
    bias = torch.tensor(v, dtype=torch.float32, device=DEV)
    a, w = torch.zeros(rows, 64, device=DEV), torch.zeros(len(v), 64, device=DEV)
    out = B.dit_linear(a, w, bias, act=1).cpu().double()
    x = bias.cpu().double()
    ref = torch.nn.functional.gelu(x, approximate="tanh")
    assert torch.equal(torch.isnan(out), torch.isnan(ref).expand(rows, -1))
    assert (out[:, v == np.inf] == np.inf).all()
    m = torch.isfinite(ref)
    bound = 8 * 2.0 ** -24 * torch.maximum(ref.abs(), x.abs().clamp(max=14) / 8)[m] + 1e-36
    assert ((out[:, m] - ref[m]).abs() <= bound).all()


def gelu64(x):
    """tanh-form GELU in float64 as x / (1 + exp(-2u)), which does not cancel in the negative tail."""
    return x / (1 + np.exp(np.minimum(-2 * math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3), 700)))


def gelu_alone(values, rows=1):
    """The fp32 GELU epilogue on `values`: zero product, the value in the bias."""
    bias = torch.tensor(values, dtype=torch.float32, device=DEV)
    return B.dit_linear(torch.zeros(rows, 64, device=DEV), torch.zeros(len(values), 64, device=DEV), bias, act=1).cpu().double().numpy()


@pytest.mark.parametrize("rows", [1, 64])
def test_fp32_gelu_of_large_negative_arguments(rows):
    """Zero, not a fraction of the argument; and down to where it vanishes as good as its exponent: t = -2u log2(e) is rounded
    two or three times, 2^-24 * |t| of the result each at most, everything else a few roundings more."""
    far = [-11.0, -1e2, -1e4, -3e18, -1e19, -1e31, -1e38, -np.finfo(np.float32).max]
    out = gelu_alone(np.concatenate([far, [0.0] * 4]), rows)
    assert (out == 0).all(), out[0]
    x = np.linspace(-10, -0.5, 764).astype(np.float32).astype(np.float64)
    t = 2 * math.sqrt(2 / math.pi) * np.abs(x + 0.044715 * x ** 3) / math.log(2)
    out, ref = gelu_alone(x, rows), gelu64(x)
    assert (np.abs(out - ref) <= 2.0 ** -24 * (4 + 3 * t) * np.abs(ref) + 1e-37).all()
    assert np.isnan(gelu_alone([-np.inf, np.nan, 0, 0])[0, :2]).all()


def test_fp32_gelu_is_as_good_as_the_tanh_form():
    """Error against float64 over N(0, 1) and wider.  0.5 x (1 + tanh(u)) in fp32 with a correctly rounded tanh has 3.80e-8 of the
    result's norm at one standard deviation, 4.05e-8 at a quarter and 2.80e-8 at three."""
    rng = np.random.default_rng(5)
    for scale, bound in ((1.0, 3.80e-8), (0.25, 4.05e-8), (3.0, 2.80e-8)):
        x = (scale * rng.standard_normal(200000)).astype(np.float32).astype(np.float64)
        err = rel(gelu64(x), gelu_alone(x)[0])
        print(scale, err, flush=True)
        assert err <= bound, (scale, err)


def as_scores(scores, head_dim):
    """q, k [1, N, 1, d] whose scores at scale 1 are scores[j] for every query: one product that is not zero, of 2^40 and a
    multiple of 2^-40."""
    n = len(scores)
    q, k = torch.zeros(1, n, 1, head_dim, device=DEV), torch.zeros(1, n, 1, head_dim, device=DEV)
    q[..., 5] = 2.0 ** 40
    k[0, :, 0, 5] = torch.tensor(np.asarray(scores, np.float32) * np.float32(2.0 ** -40), device=DEV)
    return q, k


@pytest.mark.parametrize("d", [16, 32, 64])
@pytest.mark.parametrize("n", [9, 64, 130])
def test_attention_fp32_of_scores_near_the_end_of_the_range(d, n):
    """Finite scores beyond the largest number over log2(e) (2.36e38), of either sign: differences are huge or zero, so the
    result is the value of the largest score's key, or the mean of two."""
    rng = np.random.default_rng(n)
    v = torch.randn(1, n, 1, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(n))
    for top, rest in ((3e38, 2.5e38), (3e38, -3e38), (-2.9e38, -3.2e38), (2.4e38, 0.0), (-2.4e38, -3.3e38)):
        at = rng.permutation(n)[:2]
        for winners in (at[:1], at):
            s = np.full(n, rest)
            s[winners] = top
            q, k = as_scores(s, d)
            out = B.attn3d(q, k, v, 1.0)[0, :, 0]
            want = v[0, winners, 0].double().mean(0).float().expand(n, d)
            assert torch.equal(out, want), (top, rest, winners)


@pytest.mark.parametrize("seed", [0, 1])
def test_attention_fp32_probabilities_one_by_one(seed):
    """Values that are the unit vectors: the result is the probabilities.  Scores whose differences are exact, down to 87 below
    the largest, where exp(-87) is the smallest normal number.  An exponential of one unit in the last place (2^-23 of it at
    most), 18 roundings of the key sum, one each of the products with 1 and of the division: 12 * 2^-23."""
    rng = np.random.default_rng(seed)
    s = -np.round(rng.uniform(0, 87, 64) * 1024) / 1024
    s[rng.integers(64)] = 0.0
    q, k = as_scores(s, 64)
    out = B.attn3d(q, k, torch.eye(64, device=DEV)[None, :, None], 1.0)[0, :, 0].double().cpu().numpy()
    e = np.exp(s)
    ref = np.broadcast_to(e / e.sum(), out.shape)
    assert (np.abs(out - ref) <= 12 * 2.0 ** -23 * ref).all(), np.max(np.abs(out - ref) / ref)


@pytest.mark.parametrize("n", [64, 128, 200])
def test_attention_fp32_keeps_probabilities_below_the_normal_range(n):
    """Weights of 2^-127 to 2^-149 on values of 1e30, in a tile with nothing else that is far and behind others: two units of
    2^-149, and a few roundings."""
    for far in ([-88.0], [-88.0, -92.0, -100.0]):
        s = np.zeros(n)
        s[7:7 + len(far)] = far
        q, k = as_scores(s, 64)
        v = torch.zeros(1, n, 1, 64, device=DEV)
        for i in range(len(far)):
            v[0, 7 + i, 0, i] = 1e30
        out = B.attn3d(q, k, v, 1.0)[0, :, 0, :len(far)].double().cpu().numpy() * (n - len(far))
        ref = np.exp(np.asarray(far)) * 1e30
        assert (np.abs(out - ref) <= 2 * 2.0 ** -149 * 1e30 + 1e-6 * ref).all(), (far, out[0], ref)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_narrow_network_of_scores_near_the_end_of_the_range(sign):
    """Queries and keys of the first head from their biases alone, turned by their frame: scores of 3.2e38 times the cosine of
    the distance in frames, equal within a frame.  Against the oracle and the kernels of an operation each."""
    cfg = I.CONFIGS["tiny_text"].with_(layers=2, frames=2, height=8, width=8, text_tokens=0)
    W = [(name, np.array(w)) for name, w in I.make_weights(cfg, 1001, "unit")]
    hd = cfg.head_dim
    for name, w in W:
        if name.startswith("b_qkv."):
            w[0], w[cfg.hidden] = np.float32(1e19) * np.float32(hd ** 0.5), np.float32(sign * 3.2e19)
    d = B.dit_create(cfg, B.weights_to_device(cfg, W, DEV))
    x = I.make_latent(cfg, 1)
    eps = B.dit_forward(d, torch.from_numpy(x).to(DEV), None, [500]).clone()
    assert torch.isfinite(eps).all()
    assert O.rel_mae(O.dit_forward(cfg, dict(W), x, None, [500]), eps.cpu().numpy())[2] <= 1e-5
    B.dit_set_kernel_path(d, 1)
    assert O.rel_mae(eps.cpu().numpy(), B.dit_forward(d, torch.from_numpy(x).to(DEV), None, [500]).cpu().numpy())[2] <= 1e-5

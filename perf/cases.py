"""Performance cases: the work a serving program has this framework do.

Each case is one call (or one request's chain of calls) through the package's public entry
points, on inputs made from a seed, with the bytes and operations it cannot do without, a
tolerance, and the same result from plain torch in float64.

What the ranges stand for
  lookup     a batch of prompt embeddings against the vector DB: from a test-sized float32
             cache to 10 M bfloat16 rows, one request or a batch of 256
  ivf        the same through the IVF index, for single requests over large caches
  linear, conv, attention
             single layers at the shapes a latent-diffusion UNet gives them (SD-1.5 and SDXL
             channel counts, one image to batches of eight with guidance, other resolutions,
             channel counts off the usual grid)
  eps        one UNet evaluation (guidance rows of every sample)
  denoise    the guided DDIM steps that remain after a cache hit, every sample at its own K
  request    one small request whole: lookup, state fetch, K to the host, denoise
"""
import math

import torch

import paper_2312_04429_amd as nv

THRESHOLDS = (0.95, 0.90, 0.85, 0.75, 0.65)  # the paper's selector
SKIPS = (25, 20, 15, 10, 5)
SCHED = (1000, 50, 0.00085, 0.012)           # T, N, beta range
GUIDANCE = 7.5

NETS = {
    "tiny": dict(in_ch=4, out_ch=4, H=16, W=16, ch=(32, 64), depth=(0, 1), mid_depth=1, n_res=1,
                 n_heads=4, head_dim=0, gn_groups=8, ctx_len=8, ctx_dim=64, pooled_dim=0,
                 gn_eps=1e-5, ln_eps=1e-5),
    "sd15": dict(in_ch=4, out_ch=4, H=64, W=64, ch=(320, 640, 1280, 1280), depth=(1, 1, 1, 0),
                 mid_depth=1, n_res=2, n_heads=8, head_dim=0, gn_groups=32, ctx_len=77,
                 ctx_dim=768, pooled_dim=0, gn_eps=1e-5, ln_eps=1e-5),
}


def listed():
    return [
        # the smallest request, end to end: launches and host latency are all there is
        dict(name="request_tiny", kind="request", net="tiny", n=1024, d=64, steps=20),
        # a single request against an ordinary cache: one embedding, 100 k prompts
        dict(name="lookup_100k", kind="lookup", n=100_000, d=768, m=1, dtype="bf16"),
        # a serving batch of eight against a large cache
        dict(name="lookup_1m", kind="lookup", n=1_000_000, d=768, m=8, dtype="bf16"),
        # the retrieval-heavy batch: 256 embeddings against 10 M prompts
        dict(name="lookup_10m", kind="lookup", n=10_000_000, d=768, m=256, dtype="bf16"),
        # embeddings kept as they come, in float32, at the paper's 300 k prompts
        dict(name="lookup_f32_300k", kind="lookup", n=300_000, d=768, m=4, dtype="f32"),
        # one request through the index over a million prompts
        dict(name="ivf_1m", kind="ivf", n=1_000_000, d=768, m=1, dtype="bf16", lists=1024,
             probe=32),
        # SDXL level 2 feed-forward output, batch of two with guidance
        dict(name="linear_sdxl_ff2", kind="linear", M=4096, N=1280, K=5120, K2=0, res=True),
        # SD-1.5 level 1 ResBlock convolution, batch of eight with guidance
        dict(name="conv_sd15_b8", kind="conv", B=16, H=32, W=32, C1=640, C2=0, Co=640, stride=1,
             up=False),
        # SD-1.5 level 0 self-attention, one image with guidance: 40-wide heads
        dict(name="attn_sd15_l0", kind="attention", rows=2, S=4096, L=4096, heads=8, dh=40),
        # SDXL level 1 self-attention, batch of two with guidance: 64-wide heads
        dict(name="attn_sdxl_l1", kind="attention", rows=4, S=4096, L=4096, heads=10, dh=64),
        # one evaluation of the SD-1.5-shaped network for one image
        dict(name="eps_sd15_b1", kind="eps", net="sd15", B=1),
        # eight requests that resume at different K, the last steps of each
        dict(name="denoise_sd15_b8", kind="denoise", net="sd15", B=8, left="6,5,4,4,3,3,2,2"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("lookup", "lookup", "lookup", "ivf", "linear", "linear", "conv", "conv",
                       "attention", "attention", "eps", "denoise", "request"))
    if kind == "lookup":
        c = dict(kind=kind, n=_log(rng, 500, 4_000_000), d=rng.choice((64, 384, 512, 768, 768, 1024)),
                 m=_log(rng, 1, 256), dtype=rng.choice(("bf16", "bf16", "f32")))
        if c["dtype"] == "f32":
            c["n"], c["m"] = min(c["n"], 1_000_000), min(c["m"], 32)
        return c
    if kind == "ivf":
        return dict(kind=kind, n=_log(rng, 20_000, 2_000_000), d=rng.choice((384, 768)),
                    m=_log(rng, 1, 16), dtype=rng.choice(("bf16", "bf16", "f32")),
                    lists=rng.choice((256, 1000, 1024)), probe=rng.randint(4, 64))
    side = lambda: 8 * rng.randint(4, 12)  # latent sides of 256 to 768 pixel images
    if kind == "linear":
        C = rng.choice((320, 640, 1280, 1280, 384, 200))
        form = rng.choice(("proj", "qkv", "ff2", "skip", "ctx"))
        lv = rng.choice((1, 2, 4))
        M = rng.choice((2, 4, 8, 16)) * (side() // lv) * (side() // lv)
        if form == "ctx":
            return dict(kind=kind, M=77 * rng.randint(2, 16), N=2 * C, K=rng.choice((768, 2048)),
                        K2=0, res=False)
        N, K, K2 = {"proj": (C, C, 0), "qkv": (3 * C, C, 0), "ff2": (C, 4 * C, 0),
                    "skip": (C, C, C)}[form]
        return dict(kind=kind, M=min(M, 65536), N=N, K=K, K2=K2, res=form in ("proj", "ff2"))
    if kind == "conv":
        C = rng.choice((320, 640, 1280, 256, 72))
        lv = rng.choice((1, 2, 4)) if C < 1280 else rng.choice((4, 8))
        h, w = side() // lv, side() // lv
        form = rng.choice(("same", "same", "concat", "down", "up"))
        if form == "down":
            h, w = h + h % 2, w + w % 2
        if form == "up":
            h, w = max(1, h // 2), max(1, w // 2)
        return dict(kind=kind, B=rng.choice((2, 4, 8)), H=h, W=w, C1=C,
                    C2=C if form == "concat" else 0, Co=C, stride=2 if form == "down" else 1,
                    up=form == "up")
    if kind == "attention":
        dh, heads, lv = rng.choice(((40, 8, 1), (80, 8, 2), (160, 8, 4), (64, 10, 1), (64, 20, 2)))
        S = (side() // lv) * (side() // lv)
        return dict(kind=kind, rows=rng.choice((2, 4, 6)), S=S, L=rng.choice((S, S, 77)),
                    heads=heads, dh=dh)
    if kind == "eps":
        return dict(kind=kind, net="sd15", B=rng.randint(2, 6))
    if kind == "denoise":
        B = rng.randint(1, 6)
        return dict(kind=kind, net="sd15", B=B,
                    left=",".join(str(rng.randint(1, 4)) for _ in range(B)))
    return dict(kind=kind, net="tiny", n=_log(rng, 300, 20_000), d=64, steps=rng.choice((20, 50)))


# ------------------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _cache(g, n, d, dtype):
    """Prompt embeddings: unit rows around n / 1000 themes."""
    themes = _unit(_randn(g, max(16, n // 1000), d))
    out = torch.empty(n, d, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                      device="cuda")
    for a in range(0, n, 262144):
        b = min(n, a + 262144)
        t = torch.randint(0, themes.shape[0], (b - a,), generator=g, device="cuda")
        out[a:b] = _unit(themes[t] + 0.05 * _randn(g, b - a, d))
    return out


def _queries(g, cache, m):
    """Half rewordings of cached prompts (cosine 0.6 to 0.99), half unrelated prompts."""
    n, d = cache.shape
    near = _unit(cache[torch.randint(0, n, (m,), generator=g, device="cuda")].float())
    s = 0.6 + 0.39 * torch.rand(m, 1, generator=g, device="cuda")
    u = _randn(g, m, d)
    u = _unit(u - (u * near).sum(1, keepdim=True) * near)
    q = s * near + (1 - s * s).sqrt() * u
    if m > 1:
        q[m // 2:] = _unit(_randn(g, m - m // 2, d))
    return q.contiguous()


def _params(cfg):
    """(name, shape) of every parameter in the order of the weight blob."""
    out, c0, levels = [], cfg["ch"][0], len(cfg["ch"])
    td = 4 * c0
    norm = lambda n, c: out.extend([(n + ".g", (c,)), (n + ".b", (c,))])
    conv = lambda n, o, i: out.extend([(n + ".w", (o, i, 3, 3)), (n + ".b", (o,))])

    def lin(n, o, i, bias=True):
        out.append((n + ".w", (o, i)))
        if bias:
            out.append((n + ".b", (o,)))

    def res(n, ci, co):
        norm(n + ".gn1", ci)
        conv(n + ".conv1", co, ci)
        lin(n + ".temb", co, td)
        norm(n + ".gn2", co)
        conv(n + ".conv2", co, co)
        if ci != co:
            lin(n + ".skip", co, ci)

    def tr(n, c, depth):
        norm(n + ".gn", c)
        lin(n + ".proj_in", c, c)
        for j in range(depth):
            b = f"{n}.blk{j}"
            norm(b + ".ln1", c)
            for p in "qkv":
                lin(f"{b}.attn1.{p}", c, c, False)
            lin(b + ".attn1.o", c, c)
            norm(b + ".ln2", c)
            lin(b + ".attn2.q", c, c, False)
            lin(b + ".attn2.k", c, cfg["ctx_dim"], False)
            lin(b + ".attn2.v", c, cfg["ctx_dim"], False)
            lin(b + ".attn2.o", c, c)
            norm(b + ".ln3", c)
            lin(b + ".ff1", 8 * c, c)
            lin(b + ".ff2", c, 4 * c)
        lin(n + ".proj_out", c, c)

    lin("time.l1", td, c0)
    lin("time.l2", td, td)
    conv("conv_in", c0, cfg["in_ch"])
    skips, cur = [c0], c0
    for lv, co in enumerate(cfg["ch"]):
        for r in range(cfg["n_res"]):
            res(f"down{lv}.res{r}", cur, co)
            cur = co
            if cfg["depth"][lv]:
                tr(f"down{lv}.attn{r}", cur, cfg["depth"][lv])
            skips.append(cur)
        if lv < levels - 1:
            conv(f"down{lv}.ds", cur, cur)
            skips.append(cur)
    res("mid.res0", cur, cur)
    if cfg["mid_depth"]:
        tr("mid.attn", cur, cfg["mid_depth"])
    res("mid.res1", cur, cur)
    for lv in reversed(range(levels)):
        for r in range(cfg["n_res"] + 1):
            res(f"up{lv}.res{r}", cur + skips.pop(), cfg["ch"][lv])
            cur = cfg["ch"][lv]
            if cfg["depth"][lv]:
                tr(f"up{lv}.attn{r}", cur, cfg["depth"][lv])
        if lv:
            conv(f"up{lv}.us", cur, cur)
    norm("out.gn", cur)
    conv("conv_out", cfg["out_ch"], cur)
    return out


def _weights(cfg):
    """The flat weight blob on the GPU (bfloat16 values in float32) and its parameters."""
    ps = _params(cfg)
    total = sum(math.prod(s) for _, s in ps)
    flat = (0.02 * _randn(_gen(1), total)).bfloat16().float()
    at, where = 0, {}
    for name, shape in ps:
        k = math.prod(shape)
        where[name] = flat[at:at + k].view(shape)
        if name.endswith(".g"):
            where[name].copy_((1 + where[name]).bfloat16().float())
        at += k
    return flat, where


_handles = {}


def _net(name):
    """The served model: created once, as a server does, whatever requests come."""
    if name not in _handles:
        flat, _ = _weights(NETS[name])
        _handles[name] = nv.NvUNet(NETS[name], flat.cpu().numpy())
    return _handles[name]


def _contexts(g, B, cfg):
    return _randn(g, B, cfg["ctx_len"], cfg["ctx_dim"]).bfloat16().float()


def prepare(case, seed):
    g, k, half = _gen(seed), case["kind"], torch.float16
    if k in ("lookup", "ivf"):
        cache = _cache(g, case["n"], case["d"], case["dtype"])
        s = dict(case=case, cache=cache, q=_queries(g, cache, case["m"]))
        if k == "ivf":
            init = torch.randperm(case["n"], generator=g, device="cuda")[:case["lists"]]
            s["index"] = nv.NvIVF(cache, init.cpu().numpy(), iters=1)
        return s
    if k == "linear":
        M, N, K, K2 = case["M"], case["N"], case["K"], case["K2"]
        return dict(case=case, x=_randn(g, M, K).to(half),
                    x2=_randn(g, M, K2).to(half) if K2 else None,
                    w=(0.02 * _randn(g, N, K + K2)).to(half), b=0.02 * _randn(g, N),
                    r=_randn(g, M, N).to(half) if case["res"] else None)
    if k == "conv":
        B, H, W, C1, C2, Co = (case[n] for n in ("B", "H", "W", "C1", "C2", "Co"))
        return dict(case=case, x=_randn(g, B, H, W, C1).to(half),
                    x2=_randn(g, B, H, W, C2).to(half) if C2 else None,
                    w=(0.02 * _randn(g, Co, 3, 3, C1 + C2)).to(half), b=0.02 * _randn(g, Co))
    if k == "attention":
        rows, S, L, C = case["rows"], case["S"], case["L"], case["heads"] * case["dh"]
        Lp = (L + 7) // 8 * 8
        vt = torch.zeros(C, rows, Lp, dtype=half, device="cuda")
        vt[:, :, :L] = _randn(g, C, rows, L).to(half)
        return dict(case=case, q=_randn(g, rows, S, C).to(half), k=_randn(g, rows, L, C).to(half),
                    vt=vt.view(C, rows * Lp), Lp=Lp)
    cfg, net = NETS[case["net"]], _net(case["net"])
    B = case.get("B", 1)
    s = dict(case=case, net=net, cond=_contexts(g, B, cfg), uncond=_contexts(g, B, cfg),
             x=_randn(g, B, cfg["in_ch"], cfg["H"], cfg["W"]))
    if k == "eps":
        s["step"] = [(7 * seed + 11 * b) % SCHED[1] for b in range(B)]
    elif k == "denoise":
        s["k"] = [SCHED[1] - int(v) for v in case["left"].split(",")]
    else:  # a hit: the prompt rewords a cached one, whose states after 5 and 10 steps are kept
        s["cache"] = _cache(g, case["n"], case["d"], "f32")
        s["q"] = _queries(g, s["cache"], 1)
        s["store"] = _randn(g, case["n"], 2, cfg["in_ch"], cfg["H"], cfg["W"])
        s["payload"] = torch.randperm(case["n"], generator=g, device="cuda").int()
    return s


# ------------------------------------------------------------------------------ the pass

def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "lookup":
        return nv.nv_cache_lookup(s["q"], s["cache"], THRESHOLDS, SKIPS)
    if k == "ivf":
        return s["index"].search(s["q"], c["probe"], THRESHOLDS, SKIPS)
    if k == "linear":
        return nv.nv_op_linear(s["x"], s["w"], s["b"], s["r"], x2=s["x2"])
    if k == "conv":
        return nv.nv_op_conv3x3(s["x"], s["w"], s["b"], stride=c["stride"], upsample=c["up"],
                                x2=s["x2"])
    if k == "attention":
        return nv.nv_op_attention(s["q"], s["k"], s["vt"], c["heads"], c["dh"] ** -0.5, L=c["L"],
                                  vt_row=s["Lp"])
    if k == "eps":
        return s["net"].nv_unet_eps(s["x"], s["step"], s["cond"], s["uncond"], sched=SCHED)
    if k == "denoise":
        return s["net"].nv_denoise(s["x"].clone(), s["k"], s["cond"], s["uncond"],
                                   guidance=GUIDANCE, sched=SCHED)
    idx, sim, kk = nv.nv_cache_lookup(s["q"], s["cache"], (0.90, 0.75), (10, 5))
    x = nv.nv_gather_states(s["store"], (10, 5), s["payload"], c["n"], idx, kk, s["x"])
    x = s["net"].nv_denoise(x, kk.tolist(), s["cond"], s["uncond"], guidance=GUIDANCE,
                            sched=(SCHED[0], c["steps"]) + SCHED[2:])
    return idx, sim, kk, x


# ------------------------------------------------------------------------------ its work

def _net_work(cfg, B):
    """Operations of one evaluation on 2 B guidance rows, and the bytes of its weights."""
    H, W, td = cfg["H"], cfg["W"], 4 * cfg["ch"][0]
    heads = lambda c: cfg["n_heads"] or c // cfg["head_dim"]
    flops = 0.0
    where = {}
    for lv in range(len(cfg["ch"])):
        where[f"down{lv}"] = where[f"up{lv}"] = (H >> lv) * (W >> lv)
    where["mid"] = where[f"down{len(cfg['ch']) - 1}"]
    for name, shape in _params(cfg):
        if len(shape) < 2 or ".attn2.k" in name or ".attn2.v" in name or name.startswith("time."):
            continue
        hw = where.get(name.split(".")[0], H * W)
        if ".temb" in name:
            hw = 1
        elif ".ds" in name:
            hw //= 4
        elif ".us" in name:
            hw *= 4
        flops += 2.0 * math.prod(shape) * hw
        if name.endswith(".attn1.q.w"):  # scores and their products, self and cross
            flops += 4.0 * hw * (hw + cfg["ctx_len"]) * shape[0]
    return 2 * B * flops, 2.0 * sum(math.prod(s) for _, s in _params(cfg))


def work(case):
    c, k = case, case["kind"]
    if k in ("lookup", "ivf"):
        e = 2 if c["dtype"] == "bf16" else 4
        rows = c["n"] if k == "lookup" else c["lists"] + c["m"] * c["probe"] * c["n"] // c["lists"]
        each = c["m"] if k == "lookup" else 1
        per = c["m"] * c["lists"] if k == "ivf" else 0
        return dict(bytes=rows * c["d"] * e + c["m"] * (c["d"] * 4 + 16),
                    flops=2.0 * c["d"] * (rows * each + per))
    if k == "linear":
        K = c["K"] + c["K2"]
        return dict(bytes=2.0 * (c["M"] * K + c["N"] * K + c["M"] * c["N"] * (2 if c["res"] else 1)),
                    flops=2.0 * c["M"] * c["N"] * K)
    if k == "conv":
        C = c["C1"] + c["C2"]
        px = c["B"] * c["H"] * c["W"]
        out = px * 4 if c["up"] else px // c["stride"] ** 2
        return dict(bytes=2.0 * (px * C + 9 * C * c["Co"] + out * c["Co"]),
                    flops=2.0 * out * 9 * C * c["Co"])
    if k == "attention":
        C = c["heads"] * c["dh"]
        return dict(bytes=2.0 * c["rows"] * C * 2 * (c["S"] + c["L"]),
                    flops=4.0 * c["rows"] * c["S"] * c["L"] * C)
    cfg = NETS[c["net"]]
    flops, weights = _net_work(cfg, 1)
    if k == "eps":
        return dict(bytes=weights, flops=c["B"] * flops)
    if k == "denoise":
        left = [int(v) for v in c["left"].split(",")]
        return dict(bytes=weights * max(left), flops=flops * sum(left))
    steps = c["steps"] - 10  # a hit at the higher K
    return dict(bytes=weights * steps + 4.0 * c["n"] * c["d"], flops=flops * steps)


def tolerance(case):
    k = case["kind"]
    if k in ("lookup", "ivf"):
        return "exact"  # the canonical float64 score decides: rows, similarities and K to the bit
    # four times the distance from float64 measured over these ranges: 2.1e-4 for the float16
    # results of single layers, 3.6e-4 with float16 probabilities, 1.6e-3 for an evaluation of
    # the SD-1.5 network and 1.0e-3 / 6e-4 for the latents after several steps
    rel = dict(linear=8e-4, conv=8e-4, attention=1.5e-3, eps=6e-3, denoise=4e-3, request=2.5e-3)[k]
    return dict(rel=rel, max=10 * rel)


# ------------------------------------------------------------------------------ float64

def _lookup64(s, q, cache, thresholds, skips):
    q = q.double()
    best = torch.full((q.shape[0],), -math.inf, dtype=torch.float64, device="cuda")
    at = torch.zeros(q.shape[0], dtype=torch.int64, device="cuda")
    for a in range(0, cache.shape[0], 131072):
        v, i = (q @ cache[a:a + 131072].double().T).max(dim=1)
        new = v > best
        best, at = torch.where(new, v, best), torch.where(new, i + a, at)
    kk = torch.zeros_like(at)
    for t, skip in reversed(list(zip(thresholds, skips))):
        kk = torch.where(best.float() > t, torch.full_like(kk, skip), kk)
    return at, best, kk


def _ivf64(s):
    """The best row of the probed lists, by the index's own lists."""
    c, ix = s["case"], s["index"]
    q = s["q"].double()
    order = (q @ ix.cents.double().T).topk(c["probe"], dim=1).indices.tolist()
    off = ix.offsets.tolist()
    best, at = [], []
    for j, lists in enumerate(order):
        perm = torch.cat([ix.perm[off[l]:off[l + 1]] for l in lists])
        v, i = (s["cache"][perm].double() @ q[j]).max(dim=0)
        best.append(v)
        at.append(perm[i])
    return torch.stack(at), torch.stack(best)


def _conv64(x, w, b, stride=1):
    """x [B][H][W][C], w [Co][C][3][3]."""
    B, H, W, C = x.shape
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    p = torch.zeros(B, H + 2, W + 2, C, dtype=x.dtype, device=x.device)
    p[:, 1:-1, 1:-1] = x
    out = b.expand(B * Ho * Wo, -1).clone()
    for ky in range(3):
        for kx in range(3):
            a = p[:, ky:ky + stride * (Ho - 1) + 1:stride, kx:kx + stride * (Wo - 1) + 1:stride]
            out.addmm_(a.reshape(-1, C), w[:, :, ky, kx].T.contiguous())
    return out.view(B, Ho, Wo, -1)


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2)


def _attn64(q, k, v, heads):
    """q [B][S][C], k, v [B][L][C]."""
    B, S, C = q.shape
    split = lambda t: t.reshape(-1, heads, C // heads).transpose(0, 1).contiguous()
    out = torch.empty_like(q)
    for b in range(B):
        qb, kb, vb = split(q[b]), split(k[b]), split(v[b])
        for h in range(heads):
            p = torch.softmax(qb[h] @ kb[h].T.contiguous() * (C // heads) ** -0.5, dim=-1)
            out[b, :, h * (C // heads):(h + 1) * (C // heads)] = p @ vb[h]
    return out


class _Net64:
    """The network in float64, activations [rows][H][W][C]."""

    def __init__(self, cfg):
        self.cfg = cfg
        self.flat, self.w = _weights(cfg)

    def p(self, n):
        return self.w[n].double()

    def lin(self, x, n, bias=True):
        y = x @ self.p(n + ".w").T
        return y + self.p(n + ".b") if bias else y

    def conv(self, x, n, stride=1):
        return _conv64(x, self.p(n + ".w"), self.p(n + ".b"), stride)

    def gn(self, x, n):
        G = self.cfg["gn_groups"]
        B, H, W, C = x.shape
        y = x.reshape(B, H * W, G, C // G)
        d = y - y.mean(dim=(1, 3), keepdim=True)
        y = d / (d.square().mean(dim=(1, 3), keepdim=True) + self.cfg["gn_eps"]).sqrt()
        return y.reshape(x.shape) * self.p(n + ".g") + self.p(n + ".b")

    def ln(self, x, n):
        d = x - x.mean(-1, keepdim=True)
        y = d / (d.square().mean(-1, keepdim=True) + self.cfg["ln_eps"]).sqrt()
        return y * self.p(n + ".g") + self.p(n + ".b")

    def res(self, x, temb, n):
        silu = torch.nn.functional.silu
        h = self.conv(silu(self.gn(x, n + ".gn1")), n + ".conv1")
        h = h + self.lin(silu(temb), n + ".temb")[:, None, None]
        h = self.conv(silu(self.gn(h, n + ".gn2")), n + ".conv2")
        return h + (self.lin(x, n + ".skip") if n + ".skip.w" in self.w else x)

    def tr(self, x, ctx, n, depth):
        B, H, W, C = x.shape
        heads = self.cfg["n_heads"] or C // self.cfg["head_dim"]
        h = self.lin(self.gn(x, n + ".gn").view(B, H * W, C), n + ".proj_in")
        for j in range(depth):
            b = f"{n}.blk{j}"
            for ln, at, src in ((".ln1", ".attn1", None), (".ln2", ".attn2", ctx)):
                t = self.ln(h, b + ln)
                kv = t if src is None else src
                a = _attn64(self.lin(t, b + at + ".q", False), self.lin(kv, b + at + ".k", False),
                            self.lin(kv, b + at + ".v", False), heads)
                h = h + self.lin(a, b + at + ".o")
            a, gate = self.lin(self.ln(h, b + ".ln3"), b + ".ff1").chunk(2, dim=-1)
            h = h + self.lin(a * torch.nn.functional.gelu(gate), b + ".ff2")
        return self.lin(h, n + ".proj_out").view(x.shape) + x

    def __call__(self, x, t, ctx):
        """x [rows][C][H][W], t [rows] training steps, ctx [rows][L][D] -> eps like x."""
        cfg, c0, levels = self.cfg, self.cfg["ch"][0], len(self.cfg["ch"])
        f = torch.exp(-math.log(1e4) * torch.arange(c0 // 2, dtype=torch.float64, device="cuda")
                      / (c0 // 2))
        a = t[:, None] * f
        e = self.lin(torch.cat([a.cos(), a.sin()], 1), "time.l1")
        temb = self.lin(torch.nn.functional.silu(e), "time.l2")
        h = self.conv(x.permute(0, 2, 3, 1).contiguous(), "conv_in")
        skips = [h]
        for lv in range(levels):
            for r in range(cfg["n_res"]):
                h = self.res(h, temb, f"down{lv}.res{r}")
                if cfg["depth"][lv]:
                    h = self.tr(h, ctx, f"down{lv}.attn{r}", cfg["depth"][lv])
                skips.append(h)
            if lv < levels - 1:
                h = self.conv(h, f"down{lv}.ds", 2)
                skips.append(h)
        h = self.res(h, temb, "mid.res0")
        if cfg["mid_depth"]:
            h = self.tr(h, ctx, "mid.attn", cfg["mid_depth"])
        h = self.res(h, temb, "mid.res1")
        for lv in reversed(range(levels)):
            for r in range(cfg["n_res"] + 1):
                h = self.res(torch.cat([h, skips.pop()], -1), temb, f"up{lv}.res{r}")
                if cfg["depth"][lv]:
                    h = self.tr(h, ctx, f"up{lv}.attn{r}", cfg["depth"][lv])
            if lv:
                h = self.conv(_up(h), f"up{lv}.us")
        h = self.conv(torch.nn.functional.silu(self.gn(h, "out.gn")), "conv_out")
        return h.permute(0, 3, 1, 2)


def _denoise64(net, x, ks, cond, uncond, N):
    T, _, b0, b1 = SCHED
    t = torch.arange(T, dtype=torch.float64)
    abar = torch.cumprod(1 - (b0 ** 0.5 + (b1 ** 0.5 - b0 ** 0.5) * t / (T - 1)) ** 2, 0)
    abar = abar.float().double().tolist()  # the schedule's tables are float32
    x, B = x.double().clone(), x.shape[0]
    for i in range(min(ks), N):
        on = [b for b in range(B) if ks[b] <= i]
        ti = (N - 1 - i) * (T // N) + 1
        at, ap = abar[ti], abar[max(ti - T // N, 0)]
        tt = torch.full((len(on),), float(ti), dtype=torch.float64, device="cuda")
        eu, ec = net(x[on], tt, uncond[on].double()), net(x[on], tt, cond[on].double())
        e = eu + GUIDANCE * (ec - eu)
        x0 = (x[on] - (1 - at) ** 0.5 * e) / at ** 0.5
        x[on] = ap ** 0.5 * x0 + (1 - ap) ** 0.5 * e
    return x


def exact(case, seed):
    s, k = prepare(case, seed), case["kind"]
    if k == "lookup":
        return _lookup64(s, s["q"], s["cache"], THRESHOLDS, SKIPS)
    if k == "ivf":
        at, best = _ivf64(s)
        return at, best, None
    if k == "linear":
        x = torch.cat([s["x"], s["x2"]], 1) if case["K2"] else s["x"]
        y = x.double() @ s["w"].double().T + s["b"].double()
        return y + s["r"].double() if case["res"] else y
    if k == "conv":
        x = (torch.cat([s["x"], s["x2"]], -1) if case["C2"] else s["x"]).double()
        w = s["w"].double().permute(0, 3, 1, 2)
        return _conv64(_up(x) if case["up"] else x, w, s["b"].double(), case["stride"])
    if k == "attention":
        C = case["heads"] * case["dh"]
        v = s["vt"].view(C, case["rows"], s["Lp"])[:, :, :case["L"]].permute(1, 2, 0)
        return _attn64(s["q"].double(), s["k"].double(), v.double().contiguous(), case["heads"])
    net = _Net64(NETS[case["net"]])
    if k == "eps":
        t = torch.tensor([(SCHED[1] - 1 - i) * (SCHED[0] // SCHED[1]) + 1.0 for i in s["step"]],
                         dtype=torch.float64, device="cuda")
        return tuple(net(s["x"].double(), t, s[n].double()) for n in ("uncond", "cond"))
    if k == "denoise":
        return _denoise64(net, s["x"], s["k"], s["cond"], s["uncond"], SCHED[1])
    at, best, kk = _lookup64(s, s["q"], s["cache"], (0.90, 0.75), (10, 5))
    skip = int(kk[0])
    x = s["store"][s["payload"][at].long(), 0 if skip == 10 else 1] if skip else s["x"]
    return at, best, kk, _denoise64(net, x, [skip], s["cond"], s["uncond"], case["steps"])

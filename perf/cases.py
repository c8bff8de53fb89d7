"""Measured workloads of the library: what a decoder built on it calls, from one small sequence to full batches.

``listed()`` names them, ``draw(rng)`` gives further ones of the same ranges.  Every case goes through the binding's
entry points on buffers that ``prepare`` made, as a serving program would hold them: packed factors, cache planes in the
device layout, workspace, context, output buffers.  Entry points that advance the cache lengths are preceded by one copy
that sets the lengths back, so that a pass can be repeated on the same state.

Inputs are seeded Gaussians with the statistics the path meets: hidden states with 1 % of the channels 20 times wider,
factors scaled by 1 / sqrt(fan-in), latents with the spread such hidden states give them and an image-token prefix that
is 1.5 times wider, stored through the documented quantiser.
"""
from __future__ import annotations

import math

import torch

import paper_2604_02570_amd as W

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
OUTLIER_GAIN, OUTLIER_SHARE = 20.0, 0.01
LATENT_STD = math.sqrt(1.0 + OUTLIER_SHARE * (OUTLIER_GAIN ** 2 - 1.0))   # of x A with unit-variance columns of A
IMAGE_TOKENS, IMAGE_SIGMA = 576, 1.5
ROPE_BASE, EPS = 10000.0, 1e-5


# ------------------------------------------------------------------------------------------------ the cases
def _case(kind, batch, q_heads, kv_heads, d_head, d_model, rank, rows, latent, q="i8", **more):
    c = dict(kind=kind, batch=batch, q_heads=q_heads, kv_heads=kv_heads, d_head=d_head, d_model=d_model, rank=rank,
             rows=rows, latent=latent, q=q, ragged=False, layers=1, page_rows=0, tokens=0, ffn=0)
    c.update(more)
    return c


def listed():
    """The listed workloads.  `rows` counts the cached rows before the pass (the longest sequence's where ragged)."""
    return [
        # the smallest call: one sequence, short context, everything in 32 bits (a unit-test sized model, a latency floor)
        dict(_case("step", 1, 8, 8, 64, 512, 16, 256, "f32", "f32"), name="step_f32_1seq"),
        # interactive use: one sequence of a 7B-class vision-language model, image prefix plus text; 8 layers of the stack
        dict(_case("step", 1, 32, 32, 128, 4096, 32, 640, "bf16", "bf16", layers=8), name="step_bf16_1seq_8layers"),
        # batched serving of the same model with int8 latents: append + attention, 4 layers of the stack
        dict(_case("step", 16, 32, 32, 128, 4096, 32, 2047, "i8", layers=4), name="step_i8_16x2048_4layers"),
        # large ragged batch with int4 latents
        dict(_case("step", 64, 32, 32, 128, 4096, 32, 4096, "i4", ragged=True), name="step_i4_ragged_64x4096"),
        # continuous batching from a page pool, sequences of any length in shuffled pages
        dict(_case("paged", 23, 32, 32, 128, 4096, 32, 3001, "i8", ragged=True, page_rows=128), name="paged_i8_ragged_23x3001"),
        # grouped-query attention block, int4 weights and int8 activations, long context
        dict(_case("block", 32, 28, 4, 128, 3584, 64, 8191, "i8", "f32"), name="block_w4a8_gqa_32x8192"),
        # a whole quantised decoder layer from the latent query to the feed-forward output
        dict(_case("layer", 16, 32, 32, 128, 4096, 32, 2047, "i8", "f32", ffn=11008), name="layer_w4a8_16x2048"),
        # backbones with rotary position embedding: keys are formed and rotated on chip
        dict(_case("rope", 16, 32, 32, 128, 4096, 32, 2048, "i8"), name="rope_i8_16x2048"),
        # prompt: cache of all sequences built from their hidden states, then causal attention of the whole prompt
        dict(_case("prefill", 16, 32, 32, 128, 4096, 32, 0, "i8", "bf16", tokens=2048), name="prefill_i8_16x2048"),
        dict(_case("prompt", 16, 32, 32, 128, 4096, 32, 2048, "i8", "bf16", tokens=2048), name="prompt_attn_16x2048"),
        # chunked prefill: the next piece of a few prompts, odd sizes, appended behind what is cached and attended
        dict(_case("chunk", 3, 32, 32, 128, 4096, 32, 1501, "i8", "bf16", tokens=333), name="chunk_i8_3x333_after_1501"),
        # the whole-matrix scheme the method is compared with: one rank-1024 latent shared by all heads
        dict(_case("shared", 16, 32, 32, 128, 4096, 1024, 2048, "i8", "bf16"), name="shared_i8_16x2048"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more workload of the same ranges: head layouts, ranks, types and options the entry points take, batches and
    contexts spread over their logarithm, bounded by the cache size (and prompt work) of the listed ones."""
    kind = rng.choice(["step", "step", "step", "attn", "attn", "paged", "block", "layer", "rope", "prefill", "prompt", "chunk", "shared"])
    hkv, g, d, e = rng.choice([(32, 1, 128, 4096), (32, 1, 128, 4096), (8, 4, 128, 4096), (16, 2, 128, 2048), (4, 7, 128, 3584), (8, 1, 64, 512)])
    latent = rng.choice(["i8", "i8", "i8", "i4", "bf16", "f32"]) if kind in ("step", "attn") else \
        rng.choice(["i8", "i8", "i4"]) if kind in ("paged", "rope", "prefill") else "i8"
    rank = {"f32": rng.choice([16, 32, 64]), "bf16": rng.choice([16, 32, 64]), "i8": rng.choice([32, 32, 64]), "i4": 32}[latent]
    q = latent if latent in ("f32", "bf16") else rng.choice(["i8", "f32", "bf16"])
    more = {}
    if kind in ("attn", "step") and latent == "i8" and g == 1 and d == 128 and rng.random() < 0.25:
        rank = rng.choice([96, 128])
    if kind == "shared":
        hkv, g, d, e, q, rank = 32, 1, 128, 4096, "bf16", rng.choice([256, 512, 1024, 1920, 3712])
    if kind in ("block", "layer"):
        q = "f32"
        hkv, g, d, e = (4, 7, 128, 3584) if kind == "block" and rng.random() < 0.5 else (32, 1, 128, 4096)
        rank = 64 if g == 7 else 32
        more["ffn"] = rng.choice([8192, 11008, 14336]) if kind == "layer" else 0
    if kind == "rope" and g == 4:
        rank = 32
    rb = {"f32": 4.0, "bf16": 2.0, "i8": 1.0, "i4": 0.5}[latent] * rank
    heads = 1 if kind == "shared" else hkv
    batch = _log(rng, 1, 32 if kind in ("block", "layer") else 64)
    if kind in ("prefill", "prompt", "chunk"):
        q = "bf16"
        batch = _log(rng, 1, 16)
        cap = int(32768 * 2048 / (hkv * rank * (g if kind != "prefill" else 1)) / batch)
        n = _log(rng, 3, max(4, min(2048, cap // 2)))
        past = 0 if kind == "prefill" else _log(rng, 1, max(2, min(4096, cap // 2)))
        if kind == "prompt" and rng.random() < 0.4:        # a few tokens at once over a long context (verified drafts)
            n = rng.randint(1, 8)
        rows = {"prefill": 0, "chunk": past, "prompt": n + past}[kind]
        return _case(kind, batch, hkv * g, hkv, d, e, rank, rows, latent, q, tokens=n)
    rows = _log(rng, 17, 8192)
    most = 150e6 if kind != "rope" else 70e6
    if kind == "shared":
        most = 67e6 if rank <= 1024 else 40e6
    rows = max(17, min(rows, int(most / (2 * batch * heads * rb)) - 1))
    more["ragged"] = kind in ("step", "attn", "paged", "rope", "shared") and rng.random() < 0.5
    if kind == "paged":
        more["page_rows"] = rng.choice([64, 128, 256])
    return _case(kind, batch, hkv * g, hkv, d, e, rank, rows, latent, q, **more)


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _randn(g, *shape):
    return torch.randn(shape, device="cuda", generator=g, dtype=F32)


def _as(x, dtype):
    return x.to(BF16) if dtype == "bf16" else x


def _t_cap(c):
    most = c["rows"] + max(1, c["tokens"] if c["kind"] in ("prefill", "chunk") else 1)
    unit = max(64, c["page_rows"], 128 if c["kind"] == "shared" else 0)
    return (most + unit - 1) // unit * unit


def _lens(c, g):
    n = torch.full((c["layers"], c["batch"]), c["rows"], dtype=torch.int32, device="cuda")
    if c["ragged"]:
        n = torch.randint(max(1, c["rows"] // 4), c["rows"] + 1, n.shape, device="cuda", generator=g, dtype=torch.int32)
        n[:, 0] = c["rows"]
    return n


def _f16_scale(a, levels):
    s = (a / levels).to(torch.float16)
    s = torch.where(s == 0, torch.full_like(s, 2.0 ** -24), s)
    s = torch.where(torch.isinf(s), torch.full_like(s, 65504.0), s)
    return torch.where(a == 0, torch.ones_like(s), s)


def _quant8(x):
    """Symmetric int8 along the last axis: codes (as float32) and fp16 scale, the documented rounding rules."""
    s = _f16_scale(x.abs().amax(-1), 127.0)
    return torch.clamp(torch.round(x / s.float()[..., None]), -127, 127), s


def _quant4(x):
    lo, hi = torch.clamp(x.amin(-1), max=0.0), torch.clamp(x.amax(-1), min=0.0)
    s = _f16_scale(hi - lo, 15.0)
    z = torch.clamp(torch.round(-lo / s.float()), 0, 15) + 0.0
    z = torch.where(hi == lo, torch.zeros_like(z), z)
    return torch.clamp(torch.round(x / s.float()[..., None]) + z[..., None], 0, 15), s, z.to(torch.float16)


def _store_rows(x, latent):
    """fp32 latent rows -> (stored form as the import takes it, metadata or None, the values the cache then stands for)."""
    if latent == "f32":
        return x, None, x
    if latent == "bf16":
        return x.to(BF16), None, x.to(BF16).float()
    if latent == "i8":
        q, s = _quant8(x)
        return q.to(torch.int8), s, q * s.float()[..., None]
    q, s, z = _quant4(x)
    u = q.to(torch.uint8)
    return u[..., 0::2] | (u[..., 1::2] << 4), torch.stack([s, z], -1).contiguous(), (q - z.float()[..., None]) * s.float()[..., None]


def _latents(c, g, rows):
    """Cached K or V latents of one layer, [B, Hkv, rows, r] fp32 before quantisation."""
    x = _randn(g, c["batch"], c["kv_heads"], rows, c["rank"]) * LATENT_STD
    x[:, :, :IMAGE_TOKENS] *= IMAGE_SIGMA
    return x


def _spread(c, g):
    """Standard deviation of every hidden channel."""
    sig = torch.ones(c["d_model"], device="cuda")
    sig[torch.randperm(c["d_model"], device="cuda", generator=g)[: max(1, int(OUTLIER_SHARE * c["d_model"]))]] = OUTLIER_GAIN
    return sig


def _w4(g, n_out, k_in):
    """Int4 weight: codes in [-8, 7] (float32), packed nibbles, fp16 scale per output channel."""
    w = torch.clamp(torch.round(_randn(g, n_out, k_in) * 2.5), -8, 7)
    u = w.to(torch.int16).bitwise_and(15).to(torch.uint8)
    s = (k_in ** -0.5 / 2.5 * (0.75 + 0.5 * torch.rand(n_out, device="cuda", generator=g))).to(torch.float16)
    return w, u[:, 0::2] | (u[:, 1::2] << 4), s


def _inputs(c, seed):
    """Every tensor of the case before it is laid out for the library (shared by prepare and exact)."""
    g, B, Hq, Hkv, d, E, r = _gen(seed), c["batch"], c["q_heads"], c["kv_heads"], c["d_head"], c["d_model"], c["rank"]
    fdt = "f32" if c["latent"] == "f32" else "bf16"
    s = {"lens": _lens(c, g), "fdt": fdt, "layers": []}
    if c["kind"] == "shared":
        s["q"] = (_randn(g, B, Hq, d) * LATENT_STD).to(BF16)
        s["B_K"], s["B_V"] = ((_randn(g, Hq, r, d) * r ** -0.5).to(BF16) for _ in range(2))
        s["kv"] = [_store_rows(_randn(g, B, _t_cap(c), r) * LATENT_STD, "i8") for _ in range(2)]
        return s
    for _ in range(c["layers"]):
        y = {}
        y["B_K"], y["B_V"] = (_as(_randn(g, Hkv, r, d) * r ** -0.5, fdt) for _ in range(2))
        if c["kind"] in ("step", "paged", "prefill", "chunk"):
            y["A_K"], y["A_V"] = (_as(_randn(g, Hkv, E, r) * E ** -0.5, fdt) for _ in range(2))
            n = (c["tokens"],) if c["tokens"] else ()
            y["x"] = _as(_randn(g, B, *n, E) * _spread(c, g), fdt)
        if c["kind"] in ("block", "layer"):
            sig = _spread(c, g)
            y["x"] = _randn(g, B, E) * sig
            nq = Hq * d if c["kind"] == "block" else Hq * r
            y["w_in"] = _w4(g, nq + 2 * Hkv * r, E)
            y["w_out"] = _w4(g, E, nq)
            if c["kind"] == "layer":
                y["B_Q"] = (_randn(g, Hq, r, d) * r ** -0.5).to(BF16)
                y["w_gu"], y["w_d"] = _w4(g, 2 * c["ffn"], E), _w4(g, E, c["ffn"])
                y["g1"], y["g2"] = ((1.0 + 0.1 * _randn(g, E)) / sig for _ in range(2))   # trained gains damp the wide channels
        elif c["kind"] in ("prompt", "chunk"):
            y["q"] = (_randn(g, B, Hkv, c["tokens"], Hq // Hkv, d) * LATENT_STD).to(BF16)
        elif c["kind"] != "prefill":
            q = _randn(g, B, Hq, d) * LATENT_STD
            if c["q"] == "i8":
                codes, sc = _quant8(q.reshape(B, Hq * d))
                y["q"], y["q_scale"] = codes.to(torch.int8).view(B, Hq, d), sc
            else:
                y["q"] = _as(q, c["q"])
        if c["rows"]:
            y["kv"] = [_store_rows(_latents(c, g, c["rows"]), c["latent"]) for _ in range(2)]
        s["layers"].append(y)
    return s


# ------------------------------------------------------------------------------------------------ a program's state
def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    B, Hq, Hkv, d, E, r, L = c["batch"], c["q_heads"], c["kv_heads"], c["d_head"], c["d_model"], c["rank"], c["layers"]
    t_cap, dev = _t_cap(c), dict(device="cuda")
    st = {"c": c, "ctx": W.wsvd_create(0), "stream": torch.cuda.current_stream(), "t_cap": t_cap, "lens0": s["lens"], "lens": s["lens"].clone()}
    if c["kind"] == "shared":
        blocks = []
        for plane, (codes, _, _) in enumerate(s["kv"]):   # 32-token blocks, K dim-minor and V token-minor
            v = codes.view(B, t_cap // 32, 2, 16, r // 32, 2, 16) if plane else codes.view(B, t_cap // 32, 32, r // 32, 2, 16)
            v = v.permute(0, 1, 4, 2, 5, 6, 3) if plane else v.permute(0, 1, 3, 4, 2, 5)
            blocks.append(v.contiguous().view(B, -1))
        st.update(q=s["q"], B_K=s["B_K"], B_V=s["B_V"], k=blocks[0], v=blocks[1], ks=s["kv"][0][1], vs=s["kv"][1][1],
                  ws=torch.empty(W.wsvd_shared_workspace_bytes(B, Hq, d, r, t_cap), dtype=torch.uint8, **dev),
                  out=torch.zeros(B, Hq, d, **dev))
        torch.cuda.synchronize()
        return st
    x_dt = s["fdt"]
    desc = W.layer_desc(B, Hq, Hkv, d, E, r, t_cap, c["latent"], s["fdt"], x_dt, c["q"], "f32", 0.0)
    slots = c["tokens"] * Hq if c["kind"] == "prompt" and c["tokens"] * (Hq // Hkv) <= 8 else Hq
    sizes = [W.wsvd_workspace_bytes(W.layer_desc(B, slots, Hkv, d, E, r, t_cap, c["latent"], s["fdt"], x_dt, c["q"], "f32", 0.0))]
    st["ws"] = torch.empty(max(sizes), dtype=torch.uint8, **dev)
    W.wsvd_set_workspace(st["ctx"], st["ws"])
    cb, mb = W.wsvd_cache_bytes(desc)
    mb = max(mb, 16)
    st["desc"] = desc
    st["codes"] = [torch.zeros(L, cb, dtype=torch.uint8, **dev) for _ in range(2)]
    st["meta"] = [torch.zeros(L, mb // 2, dtype=torch.float16, **dev) for _ in range(2)]
    st["layers"] = []
    for l, y in enumerate(s["layers"]):
        cache = W.make_cache(st["codes"][0][l], st["codes"][1][l], st["meta"][0][l], st["meta"][1][l], st["lens"][l])
        for plane in range(2):
            if c["rows"]:
                codes, meta, _ = y["kv"][plane]
                codes = codes.contiguous()
                W.wsvd_cache_import(st["ctx"], desc, plane, codes, meta, 0, c["rows"], cache)
        n = {k: y[k].contiguous() for k in ("x", "q", "q_scale", "B_K", "B_V", "g1", "g2") if k in y}
        n["cache"] = cache
        for k in ("A_K", "A_V"):
            if k in y:
                n[k] = torch.empty(W.wsvd_factor_a_bytes(desc), dtype=torch.uint8, **dev)
                W.wsvd_pack_factor_a(st["ctx"], desc, y[k], n[k])
        for k in ("w_in", "w_out", "w_gu", "w_d"):
            if k in y:
                n[k] = y[k][1:]
        if "B_Q" in y:
            n["fold"] = torch.empty(Hq, r, r, **dev)
            W.wsvd_fold_qk(st["ctx"], desc, y["B_Q"], r, y["B_K"], n["fold"])
        st["layers"].append(n)
    if c["kind"] == "paged":
        P = c["page_rows"]
        pages = t_cap // P
        n_pages = B * pages + 3
        perm = torch.randperm(n_pages, generator=_gen(seed + 1), **dev)[: B * pages]
        st["table"] = perm.view(B, pages).to(torch.int32).contiguous()
        for name in ("codes", "meta"):
            pools = []
            for t in st[name]:
                v = t.view(B, Hkv, pages, -1)
                pool = torch.zeros(n_pages, Hkv, v.shape[-1], dtype=v.dtype, **dev)
                pool[perm] = v.permute(0, 2, 1, 3).reshape(B * pages, Hkv, -1)
                pools.append(pool)
            st[name] = pools
        st["layers"][0]["cache"] = W.make_paged_cache(*st["codes"], *st["meta"], st["lens"][0], st["table"], P, pages, n_pages)
    if c["kind"] in ("prompt", "chunk"):
        st["out"] = torch.zeros(1, B, Hkv, c["tokens"], Hq // Hkv, d, **dev)
    else:
        st["out"] = torch.zeros(L, B, Hq, d if c["kind"] != "layer" else r, **dev)
    if c["kind"] in ("block", "layer"):
        nq = Hq * (d if c["kind"] == "block" else r)
        f32, i8, f16 = (lambda dt: lambda *n: torch.zeros(*n, dtype=dt, **dev))(F32), (lambda *n: torch.zeros(*n, dtype=torch.int8, **dev)), \
            (lambda *n: torch.zeros(*n, dtype=torch.float16, **dev))
        st.update(nq=nq, xq=i8(B, E), xs=f16(B), cq=f32(B, nq), lat=f32(B, 2 * Hkv * r), uq=i8(B, nq), us=f16(B), y=f32(B, E))
        if c["kind"] == "layer":
            st.update(xr=f32(B, E), gu=f32(B, 2 * c["ffn"]), aq=i8(B, c["ffn"]), asc=f16(B), down=f32(B, E))
    torch.cuda.synchronize()
    assert W.wsvd_check(st["ctx"]) == 0
    return st


def run(st):
    c, ctx, s = st["c"], st["ctx"], st["stream"]
    kind = c["kind"]
    B, Hq, Hkv, d, E, r = c["batch"], c["q_heads"], c["kv_heads"], c["d_head"], c["d_model"], c["rank"]
    if kind == "shared":
        W.wsvd_decode_attn_shared(ctx, B, Hq, d, r, st["t_cap"], 0.0, st["q"], st["B_K"], st["B_V"], st["k"], st["v"], st["ks"], st["vs"],
                                  st["lens"], st["ws"], st["out"], s)
        return st["out"]
    desc, out = st["desc"], st["out"]
    grows = kind in ("step", "paged", "block", "layer", "prefill", "chunk")
    if grows:
        st["lens"].copy_(st["lens0"])
    for l, y in enumerate(st["layers"]):
        if kind == "step":
            W.wsvd_decode_step(ctx, desc, y["x"], None, y["A_K"], y["A_V"], y["q"], y.get("q_scale"), y["B_K"], y["B_V"], y["cache"],
                               c["rows"] + 1, out[l], s)
        elif kind == "attn":
            W.wsvd_decode_attn(ctx, desc, y["q"], y.get("q_scale"), y["B_K"], y["B_V"], y["cache"], c["rows"], out[l], s)
        elif kind == "rope":
            W.wsvd_decode_attn_rope(ctx, desc, y["q"], y.get("q_scale"), y["B_K"], y["B_V"], y["cache"], c["rows"], ROPE_BASE, out[l], s)
        elif kind == "paged":
            W.wsvd_latent_append_paged(ctx, desc, y["x"], None, y["A_K"], y["A_V"], y["cache"], s)
            W.wsvd_decode_attn_paged(ctx, desc, y["q"], y.get("q_scale"), y["B_K"], y["B_V"], y["cache"], c["rows"] + 1, out[l], s)
        elif kind == "prefill":
            W.wsvd_prefill_append(ctx, desc, y["x"], None, c["tokens"], -1, y["A_K"], y["A_V"], y["cache"], s)
        elif kind == "prompt":
            W.wsvd_prefill_attn(ctx, desc, y["q"], c["tokens"], 0, y["B_K"], y["B_V"], y["cache"], c["rows"], out[l], s)
        elif kind == "chunk":
            n = c["tokens"]
            W.wsvd_prefill_append(ctx, desc, y["x"], None, n, -1, y["A_K"], y["A_V"], y["cache"], s)
            W.wsvd_prefill_attn(ctx, desc, y["q"], n, 0, y["B_K"], y["B_V"], y["cache"], c["rows"] + n, out[l], s)
        elif kind == "block":
            nq, ld, lat = st["nq"], 2 * Hkv * r, st["lat"]
            W.wsvd_quantize_act_i8(ctx, y["x"], W.F32, B, E, st["xq"], st["xs"], s)
            W.wsvd_linear_w4a8_split(ctx, st["xq"], st["xs"], *y["w_in"], B, E, nq + ld, nq, st["cq"], lat, s)
            W.wsvd_decode_attn_store(ctx, desc, lat, lat[:, Hkv * r:], ld, st["cq"], None, y["B_K"], y["B_V"], y["cache"], c["rows"] + 1, out[l], s)
            W.wsvd_quantize_act_i8(ctx, out[l], W.F32, B, nq, st["uq"], st["us"], s)
            W.wsvd_linear_w4a8(ctx, st["uq"], st["us"], *y["w_out"], B, nq, E, st["y"], s)
        elif kind == "layer":
            nq, ld, lat, F = st["nq"], 2 * Hkv * r, st["lat"], c["ffn"]
            W.wsvd_rmsnorm_quant_i8(ctx, y["x"], None, y["g1"], EPS, B, E, None, st["xq"], st["xs"], s)
            W.wsvd_linear_w4a8_split(ctx, st["xq"], st["xs"], *y["w_in"], B, E, nq + ld, nq, st["cq"], lat, s)
            W.wsvd_latent_store(ctx, desc, lat, lat[:, Hkv * r:], ld, y["cache"], s)
            W.wsvd_decode_attn_latent(ctx, desc, st["cq"], r, y["fold"], y["cache"], c["rows"] + 1, out[l], s)
            W.wsvd_quantize_act_i8(ctx, out[l], W.F32, B, nq, st["uq"], st["us"], s)
            W.wsvd_linear_w4a8(ctx, st["uq"], st["us"], *y["w_out"], B, nq, E, st["y"], s)
            W.wsvd_rmsnorm_quant_i8(ctx, y["x"], st["y"], y["g2"], EPS, B, E, st["xr"], st["xq"], st["xs"], s)
            W.wsvd_linear_w4a8(ctx, st["xq"], st["xs"], *y["w_gu"], B, E, 2 * F, st["gu"], s)
            W.wsvd_swiglu_quant_i8(ctx, st["gu"], B, F, st["aq"], st["asc"], s)
            W.wsvd_linear_w4a8(ctx, st["aq"], st["asc"], *y["w_d"], B, F, E, st["down"], s)
    got = {} if kind == "prefill" else {"out": out}
    if grows:
        view = {"f32": F32, "bf16": BF16}.get(c["latent"], torch.uint8)
        got.update(lens=st["lens"], k_codes=st["codes"][0].view(view), v_codes=st["codes"][1].view(view))
        if c["latent"] in ("i8", "i4"):
            got.update(k_meta=st["meta"][0], v_meta=st["meta"][1])
    if kind == "block":
        got["y"] = st["y"]
    if kind == "layer":
        got.update(x_attn=st["xr"], down=st["down"])
    return got


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: the cached rows that are read (ragged: their mean), rows written, factors, weights, inputs and outputs, each
    once.  Operations: the products of the absorbed formulation (rotary: of the reconstructed keys)."""
    c = case
    B, Hq, Hkv, d, E, r, L = c["batch"], c["q_heads"], c["kv_heads"], c["d_head"], c["d_model"], c["rank"], c["layers"]
    kind, n = c["kind"], c["tokens"]
    fb = 4 if c["latent"] == "f32" else 2
    row = 2 * ({"f32": 4, "bf16": 2, "i8": 1, "i4": 0.5}[c["latent"]] * r + {"i8": 2, "i4": 4}.get(c["latent"], 0))
    rows = c["rows"] * (0.625 if c["ragged"] else 1.0)
    qb = {"i8": 1, "bf16": 2, "f32": 4}[c["q"]]
    if kind == "shared":
        return {"bytes": B * rows * row + 2 * Hq * r * d * 2 + B * Hq * d * (2 + 4), "flops": B * Hq * (4.0 * rows * r + 4.0 * r * d)}
    bytes_, flops = 0.0, 0.0
    if kind in ("step", "paged", "prefill", "chunk"):      # projection of the new tokens, their rows written
        t = max(1, n)
        bytes_ += B * t * E * fb + 2 * Hkv * E * r * fb + B * t * Hkv * row
        flops += 2.0 * B * t * E * 2 * Hkv * r
    if kind in ("step", "paged", "attn", "rope", "block", "layer"):
        bytes_ += B * rows * Hkv * row + 2 * Hkv * r * d * fb + B * Hq * d * (qb + 4)
        flops += B * Hq * (4.0 * rows * r + 4.0 * r * d) + (2.0 * B * Hq * rows * r * d if kind == "rope" else 0.0)
    if kind in ("prompt", "chunk"):
        past = c["rows"] - n if kind == "prompt" else c["rows"]
        bytes_ += B * past * Hkv * row + B * n * Hkv * row * (kind == "prompt") + 2 * Hkv * r * d * 2 + B * n * Hq * d * (2 + 4)
        flops += B * Hq * (4.0 * r * (n * past + n * (n + 1) / 2) + 4.0 * r * d * n)
    if kind in ("block", "layer"):
        nq = Hq * (d if kind == "block" else r)
        w = (nq + 2 * Hkv * r) * E + E * nq + 3 * c["ffn"] * E
        bytes_ += w / 2 + B * E * 4 * 2 + B * Hkv * row
        flops += 2.0 * B * w
    return {"bytes": L * bytes_, "flops": L * flops}


def tolerance(case):
    """Relative 2-norm, about four times what the path shows against the 64-bit result or against itself with its sums in
    another order.  32-bit sums over exactly stored latents: 5e-7 measured.  Quantised latents: 3e-6 .. 4e-6 (21-bit
    operands of the integer products); a projection summed in another order may also move a code of the new row by one
    (2 in 10^4 do), which weighs about 1 / rows.  fp16 value operands of the prompt kernels and of the shared latent: 2e-4.
    Block and layer: int8 activations are rounded again before every projection, and a 1e-6 difference moves some of them
    by one code (4e-4 after one rounding; 4e-3 to 1.3e-2 after the feed-forward, where one moved code moves hundreds).
    Whole values: codes that round the other way, 2e-5 of all new ones measured for a prompt."""
    c = case
    t_cap, new = _t_cap(c), 1.0
    rel = {"block": 1.6e-3, "layer": 3e-2, "shared": 8e-4, "prompt": 8e-4, "chunk": 8e-4, "prefill": 6e-5}.get(c["kind"])
    if rel is None:
        quantum = {"f32": 0.0, "bf16": 2e-3, "i8": 2e-3, "i4": 1.6e-2}[c["latent"]]
        rel = {"f32": 3e-6, "bf16": 3e-6, "i8": 2e-5, "i4": 3e-5}[c["latent"]] + (quantum / c["rows"] if c["kind"] in ("step", "paged") else 0.0)
    if c["kind"] not in ("prefill", "chunk"):
        new = min(1.0, 64.0 / t_cap)
    return {"rel": rel, "differ": min(0.01, 1e-4 * new + 4.0 / (c["batch"] * c["kv_heads"] * t_cap * c["rank"] / 2))}


# ------------------------------------------------------------------------------------------------ 64-bit results
def _attend(q, K, V, lens, scale):
    """softmax(scale q K^T) V per (sequence, head) in 64 bits; q [B,Hq,r], K, V [B,Hkv,T,r], rows below lens."""
    B, Hq, r = q.shape
    Hkv, T = K.shape[1:3]
    out = torch.zeros(B, Hq, V.shape[-1], dtype=F64, device="cuda")
    for b in range(B):
        n = int(lens[b])
        s = torch.matmul(K[b, :, :n].double(), q[b].view(Hkv, Hq // Hkv, r).transpose(1, 2).contiguous()) * scale
        p = torch.softmax(s, 1).transpose(1, 2).contiguous()
        out[b] = torch.matmul(p, V[b, :, :n].double()).view(Hq, -1)
    return out


def _full(c, y, t_cap):
    """Cached values [B, Hkv, t_cap, r] (fp32, exact) and metadata planes with room for the new rows."""
    B, Hkv, r = c["batch"], c["kv_heads"], c["rank"]
    vals, metas = [], []
    for plane in range(2):
        v = torch.zeros(B, Hkv, t_cap, r, device="cuda")
        m = torch.zeros(B, Hkv, t_cap, *((2,) if c["latent"] == "i4" else ()), dtype=F64, device="cuda")
        if c["rows"]:
            _, meta, val = y["kv"][plane]
            v[:, :, : c["rows"]] = val
            if meta is not None:
                m[:, :, : c["rows"]] = meta.double()
        vals.append(v)
        metas.append(m)
    return vals, metas


def _put(c, vals, metas, new, lens):
    """Rows new[plane] [B, Hkv, n, r] (64 bits) stored behind lens[b]."""
    for plane in range(2):
        _, meta, val = _store_rows(new[plane].float(), c["latent"])
        for b in range(c["batch"]):
            at, n = int(lens[b]), val.shape[2]
            vals[plane][b, :, at:at + n] = val[b]
            if meta is not None:
                metas[plane][b, :, at:at + n] = meta[b].double()


def _project(x, A):
    """[B, n, E] x [Hkv, E, r] -> [B, Hkv, n, r] in 64 bits."""
    B, n, E = x.shape
    H, _, r = A.shape
    y = x.reshape(B * n, E).double() @ A.double().permute(1, 0, 2).reshape(E, H * r)
    return y.view(B, n, H, r).permute(0, 2, 1, 3)


def _absorb(q, B_K):
    Hkv, r, d = B_K.shape
    B, Hq, _ = q.shape
    t = torch.matmul(q.double().view(B, Hkv, Hq // Hkv, d), B_K.double().transpose(1, 2).contiguous())
    return t.reshape(B, Hq, r)


def _expand(u, B_V):
    Hkv, r, d = B_V.shape
    B, Hq, _ = u.shape
    return torch.matmul(u.view(B, Hkv, Hq // Hkv, r), B_V.double()).reshape(B, Hq, d)


def _w4a8(x, w):
    q, s = _quant8(x.float())
    return (q.double() @ w[0].double().t()) * s.double()[:, None] * w[2].double()[None, :]


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    B, Hq, Hkv, d, r, kind, n = c["batch"], c["q_heads"], c["kv_heads"], c["d_head"], c["rank"], c["kind"], c["tokens"]
    scale, t_cap, got = 1.0 / math.sqrt(d), _t_cap(c), {}
    if kind == "shared":
        out = torch.zeros(B, Hq, d, dtype=F64, device="cuda")
        for b in range(B):
            t = int(s["lens"][0, b])
            K, V = (s["kv"][p][2][b, :t].double() for p in range(2))
            qt = torch.matmul(s["B_K"].double(), s["q"][b].double().unsqueeze(-1)).squeeze(-1)          # [H, R]
            u = torch.softmax(qt @ K.t() * scale, -1) @ V
            out[b] = torch.matmul(u.unsqueeze(1), s["B_V"].double()).squeeze(1)
        return out
    outs, metas_all = [], [[], []]
    for l, y in enumerate(s["layers"]):
        lens = s["lens"][l].tolist()
        (K, V), metas = _full(c, y, t_cap)
        if kind in ("step", "paged", "prefill", "chunk"):
            x = y["x"].view(B, max(1, n), -1)
            _put(c, (K, V), metas, [_project(x, y["A_K"]), _project(x, y["A_V"])], lens)
            lens = [v + max(1, n) for v in lens]
        if kind in ("block", "layer"):
            nq = Hq * (d if kind == "block" else r)
            z = _w4a8(y["x"] if kind == "block" else _rms(y["x"].double(), y["g1"]), y["w_in"])
            new = z[:, nq:].view(B, 2, Hkv, 1, r)
            _put(c, (K, V), metas, [new[:, 0], new[:, 1]], lens)
            lens = [v + 1 for v in lens]
            # (what comes after the attention is None: its int8 activations are rounded from values that differ in the
            # seventh digit, so a handful of codes fall the other way and decide how far y or down is from 64 bits)
            if kind == "block":
                o = _expand(_attend(_absorb(z[:, :nq].view(B, Hq, d), y["B_K"]), K, V, lens, scale), y["B_V"])
                got["y"] = None
            else:
                fold = torch.matmul(y["B_Q"].double(), y["B_K"].double().transpose(1, 2).contiguous().repeat_interleave(Hq // Hkv, 0))
                o = _attend(torch.matmul(z[:, :nq].view(B, Hq, 1, r), fold).view(B, Hq, r), K, V, lens, scale)
                got["x_attn"] = got["down"] = None
            outs.append(o)
        elif kind == "rope":
            theta = ROPE_BASE ** (-2.0 * torch.arange(d // 2, dtype=F64, device="cuda") / d)
            turn = lambda v, pos: (lambda a, b, co, si: torch.cat([a * co - b * si, a * si + b * co], -1))(  # noqa: E731
                v[..., : d // 2], v[..., d // 2:], torch.cos(pos[:, None] * theta), torch.sin(pos[:, None] * theta))
            q = y["q"].double() * (y["q_scale"].double()[:, None, None] if "q_scale" in y else 1.0)
            o = torch.zeros(B, Hq, d, dtype=F64, device="cuda")
            for b in range(B):
                t = lens[b]
                k = turn(torch.matmul(K[b, :, :t].double(), y["B_K"].double()), torch.arange(t, dtype=F64, device="cuda"))
                qr = turn(q[b], torch.full((Hq,), t - 1.0, dtype=F64, device="cuda")).view(Hkv, Hq // Hkv, d)
                p = torch.softmax(torch.matmul(qr, k.transpose(1, 2).contiguous()) * scale, -1)
                o[b] = torch.matmul(torch.matmul(p, V[b, :, :t].double()), y["B_V"].double()).view(Hq, d)
            outs.append(o)
        elif kind in ("step", "attn", "paged"):
            q = y["q"].double() * (y["q_scale"].double()[:, None, None] if "q_scale" in y else 1.0)
            outs.append(_expand(_attend(_absorb(q, y["B_K"]), K, V, lens, scale), y["B_V"]))
        elif kind in ("prompt", "chunk"):
            o = torch.zeros(B, Hkv, n, Hq // Hkv, d, dtype=F64, device="cuda")
            for b in range(B):
                t = lens[b]
                seen = torch.arange(t, device="cuda")[None, :] <= torch.arange(t - n, t, device="cuda")[:, None]
                for h in range(Hkv):
                    q = y["q"][b, h].double().view(-1, d) @ y["B_K"][h].double().t()
                    w = (q @ K[b, h, :t].double().t() * scale).view(n, Hq // Hkv, t).masked_fill(~seen[:, None, :], -math.inf)
                    o[b, h] = (torch.softmax(w, -1).view(-1, t) @ V[b, h, :t].double() @ y["B_V"][h].double()).view(n, Hq // Hkv, d)
            outs.append(o)
        for p in range(2):
            metas_all[p].append((metas[p] if c["latent"] in ("i8", "i4") else (K, V)[p].double()).reshape(-1))
    if kind != "prefill":
        got["out"] = torch.stack(outs)
    if kind in ("step", "block", "layer", "prefill", "chunk"):
        what = "meta" if c["latent"] in ("i8", "i4") else "codes"
        got.update({"k_" + what: torch.stack(metas_all[0]), "v_" + what: torch.stack(metas_all[1])})
    return got

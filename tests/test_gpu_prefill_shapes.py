"""Prompt projection: every kernel shape of the dispatch stores the rows the oracle's projection gives, for sizes at the
edges of its token tiles (one tile, one more, one less, several with a remainder) and sequences that already hold rows."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2604_02570_amd as W
import wsvd_inputs as WI
from cases import build_case
from harness import as_dtype_dev, check_i8_rows
from test_gpu_parity import check_out, layer_for
from test_gpu_prefill import _check_i4_rows, _latents64, _multi_q, _prefill_attn

pytestmark = pytest.mark.gpu


def _prompt(name, shape, n, **over):
    """All sequences of a small case get n more rows through kernel shape `shape`; checks them against fp64."""
    c = build_case(name, extra_cap=n + 64, **over)
    sp = c.sp
    lens = (c.cache.seq_lens // 2 * 2).astype(np.int32)     # (int4: even start rows)
    lens[0] = 0
    c.cache.seq_lens[:] = lens
    L = layer_for(c); L.upload(c.cache)
    X = np.stack([WI.bf16_exact(WI.hidden_states(sp, n, 1.0, which="ctx", sub=90 + b)) for b in range(sp.batch)])
    W.wsvd_ctx_set_option(L.ctx, "project_shape", shape)
    W.wsvd_prefill_append(L.ctx, L.desc, as_dtype_dev(X.reshape(sp.batch * n, -1), "bf16"), None, n, -1,
                          L.pack_A(c.AK, "bf16"), L.pack_A(c.AV, "bf16"), L.cache)
    assert W.wsvd_check(L.ctx) == 0
    assert (L.seq_lens.cpu().numpy() == lens + n).all()
    for b in range(sp.batch):
        for plane, A in ((0, c.AK), (1, c.AV)):
            c64, what = _latents64(X[b], A), f"{name} shape {shape} n {n} seq {b} plane {plane}"
            if sp.latent_dtype == "i4":
                _check_i4_rows(L, plane, b, int(lens[b]), n, c64, what)
            else:
                gc, gs, _ = L.download(plane, int(lens[b]), n)
                check_i8_rows(gc[b].reshape(c64.shape), gs[b].reshape(c64.shape[:-1]), c64, what)
    L.close()


@pytest.mark.parametrize("shape", [0, 1, 44])
@pytest.mark.parametrize("n", [1, 255, 257])
def test_int4_prompt_projection_shapes(shape, n):
    _prompt("c4_small", shape, n, batch=3, context=120, ragged=(60, 120))


# (the first three take 64 x 32 tiles, the fourth and the last 128 x 32, the fifth 256 x 64: channel tiles that end inside a
# workgroup's group, tokens at the edges of a tile and one sequence of several)
@pytest.mark.parametrize("name,n,over", [("c3_small", 1, dict()), ("c3_small", 33, dict(n_q_heads=7, n_kv_heads=7)), ("c3_small", 64, dict(rank=64)),
                                         ("c3_small", 345, dict(n_q_heads=32, n_kv_heads=32)), ("c3_small", 321, dict(rank=64, n_q_heads=18, n_kv_heads=18)),
                                         ("c4_small", 353, dict(n_q_heads=34, n_kv_heads=34, ragged=(60, 120)))])
def test_prompt_projection_tile_rule(name, n, over):
    _prompt(name, 0, n, **{**dict(batch=3, context=120), **over})


# the two tile kernels with hidden states through LDS keep four chunks of 64 model dims in flight: fewer chunks than that, a
# last round that is not full, and (70 tokens of 4 sequences in 64-token tiles, 40 in 32-token tiles) a number of token groups
# that is a multiple of the 8 dies
@pytest.mark.parametrize("d_model", [64, 128, 192, 320, 576])
@pytest.mark.parametrize("shape,n", [(11, 40), (22, 70), (11, 33), (22, 65)])
@pytest.mark.parametrize("name,over", [("c3_small", dict()), ("c3_small", dict(rank=64)), ("c4_small", dict(ragged=(60, 120)))], ids=["i8", "i8-r64", "i4"])
def test_prompt_projection_chunk_tails(name, over, shape, n, d_model):
    _prompt(name, shape, n, **{**dict(batch=4 if n in (40, 70) else 3, context=120, d_model=d_model), **over})


# tiles are cut from the rows of all sequences (int4: only where a sequence has an even number of tokens): several sequences in
# a tile, a tile's edge inside one; the contraction split over the wave groups of a workgroup: fewer chunks than groups, a last
# round that not every group has
@pytest.mark.parametrize("d_model", [64, 192, 448])
@pytest.mark.parametrize("shape,n", [(5, 9), (5, 34), (11, 22), (12, 21), (12, 66), (13, 22), (13, 34), (22, 22), (25, 43), (25, 130), (2, 90)])
@pytest.mark.parametrize("name,over", [("c3_small", dict()), ("c3_small", dict(rank=64)), ("c4_small", dict(ragged=(60, 120)))], ids=["i8", "i8-r64", "i4"])
def test_prompt_projection_tiles_across_sequences(name, over, shape, n, d_model):
    _prompt(name, shape, n, **{**dict(batch=4, context=120, d_model=d_model), **over})


@pytest.mark.parametrize("shape", [5, 12, 25, 2])
def test_prompt_projection_full_sequence_inside_a_tile(shape):
    """A sequence without room in the middle of a tile: reported, its own rows that fit are stored, its neighbours get theirs."""
    n = 20
    c = build_case("c3_small", batch=4, context=100, extra_cap=60)
    L = layer_for(c)
    lens = np.array([7, L.t_cap - 5, 0, 40], dtype=np.int32)
    c.cache.seq_lens[:] = lens
    L.upload(c.cache)
    X = np.stack([WI.bf16_exact(WI.hidden_states(c.sp, n, 1.0, which="ctx", sub=70 + b)) for b in range(4)])
    W.wsvd_ctx_set_option(L.ctx, "project_shape", shape)
    W.wsvd_prefill_append(L.ctx, L.desc, as_dtype_dev(X.reshape(4 * n, -1), "bf16"), None, n, -1, L.pack_A(c.AK, "bf16"), L.pack_A(c.AV, "bf16"), L.cache)
    assert W.wsvd_check(L.ctx) == W.E_CAPACITY
    assert (L.seq_lens.cpu().numpy() == np.minimum(lens + n, L.t_cap)).all()
    for b in range(4):
        m = min(n, L.t_cap - int(lens[b]))
        for plane, A in ((0, c.AK), (1, c.AV)):
            c64 = _latents64(X[b], A)[..., :m, :]
            gc, gs, _ = L.download(plane, int(lens[b]), m)
            check_i8_rows(gc[b].reshape(c64.shape), gs[b].reshape(c64.shape[:-1]), c64, f"shape {shape} seq {b} plane {plane}")
    L.close()


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("batch,n", [(64, 4), (64, 32), (16, 64), (16, 260), (1, 300), (8, 1024), (3, 333), (2, 2048), (1, 200)])
def test_prompt_projection_takes_a_fitting_tile(batch, n, rank):
    """Many short prompts, prompts just past a multiple of 256 tokens, one prompt, full batches: the tile that is taken by
    itself is about as fast as the best one asked for (a tile that does not fit the prompts costs a factor of 2 to 4)."""
    t = _tile_times(batch, n, rank, 4096)
    assert t[0] <= 1.35 * min(t.values()), t


@pytest.mark.parametrize("batch,n,rank,E", [(28, 385, 64, 192), (22, 241, 32, 320), (17, 286, 64, 64), (40, 220, 64, 320), (11, 659, 64, 512)])
def test_prompt_projection_takes_a_fitting_tile_for_a_short_contraction(batch, n, rank, E):
    """Many tokens and a small d_model: the store of the rows is a large part of the time (counted as a part of the work, the
    choice is within a tenth of the best; counted once per call it takes tiles that are 1.3 to 1.4 times slower)."""
    t = _tile_times(batch, n, rank, E)
    assert t[0] <= 1.2 * min(t.values()), t


def _tile_times(batch, n, rank, E):
    """us per call of 32 kv heads for every tile that can be asked for, and (0) for the one that is taken by itself."""
    Hkv, t_cap = 32, (n + 63) // 64 * 64
    desc = W.layer_desc(batch, Hkv, Hkv, 128, E, rank, t_cap, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
    ctx = W.wsvd_create(0)
    cb, mb = W.wsvd_cache_bytes(desc)
    codes, meta = ([torch.zeros(b, dtype=torch.uint8, device="cuda") for _ in range(2)] for b in (cb, mb))
    lens = torch.zeros(batch, dtype=torch.int32, device="cuda")
    cache = W.make_cache(*codes, *meta, lens)
    x = torch.randn(batch * n, E, device="cuda").to(torch.bfloat16)
    A = [torch.randn(W.wsvd_factor_a_bytes(desc) // 2, device="cuda").to(torch.bfloat16) for _ in range(2)]

    def us(shape):
        W.wsvd_ctx_set_option(ctx, "project_shape", shape)
        best = float("inf")
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                lens.zero_()
                W.wsvd_prefill_append(ctx, desc, x, None, n, -1, *A, cache)
            b.record(); torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        return best

    t = {shape: us(shape) for shape in (5, 11, 12, 13, 22, 25, 2, 0)}
    assert W.wsvd_check(ctx) == 0
    W.wsvd_destroy(ctx)
    return t


# query rows per kv head at the edges of the 32-row waves and of the 1 / 2 / 4 waves that share a workgroup's cache blocks;
# batch, heads, rows and key blocks choose the workgroup shape
ATTN_SHAPES = [("c3_small", 9, 0, dict()), ("c3_small", 31, 2, dict(context=700)), ("c3_small", 33, 0, dict(d_head=64, context=65)),
               ("c3_small", 65, 0, dict(batch=24, n_q_heads=8, n_kv_heads=8, context=200)),
               ("c3_small", 17, 1, dict(batch=24, n_q_heads=32, n_kv_heads=8, context=130, rank=64)),
               ("c3_small", 97, 0, dict(batch=16, n_q_heads=32, n_kv_heads=32, context=129)),
               ("c3_small", 129, 3, dict(batch=16, n_q_heads=32, n_kv_heads=32, context=161, d_head=64)),
               ("c3_small", 33, 0, dict(batch=16, n_q_heads=48, n_kv_heads=24, context=96, rank=64)),
               # one wave of rows, the key blocks dealt to 1, 2 and 4 waves: fewer blocks than waves, one more, several each
               ("c3_small", 12, 0, dict(context=20)), ("c3_small", 20, 0, dict(context=64)), ("c3_small", 20, 5, dict(context=90)),
               ("c3_small", 40, 0, dict(context=97, rank=64)), ("c3_small", 40, 1, dict(context=290, rank=64, d_head=64)),
               ("c3_small", 33, 0, dict(batch=8, n_q_heads=32, n_kv_heads=32, context=600, rank=64)),
               ("c3_small", 33, 2, dict(batch=8, n_q_heads=32, n_kv_heads=32, context=1030, rank=64)),
               ("c3_small", 33, 0, dict(batch=14, n_q_heads=32, n_kv_heads=32, context=600)),
               # a full chip: one, two and four waves of rows, full groups of four and not
               ("c3_small", 20, 0, dict(batch=40, n_q_heads=32, n_kv_heads=32, context=50, rank=64)),
               ("c3_small", 40, 0, dict(batch=36, n_q_heads=32, n_kv_heads=32, context=70)),
               ("c3_small", 40, 0, dict(batch=24, n_q_heads=32, n_kv_heads=32, context=1030, rank=64, d_head=64)),
               ("c3_small", 65, 0, dict(batch=22, n_q_heads=32, n_kv_heads=32, context=1030, d_head=64)),
               ("c3_small", 150, 0, dict(batch=16, n_q_heads=32, n_kv_heads=32, context=160))]


@pytest.mark.parametrize("name,nq,n_after,over", ATTN_SHAPES, ids=[f"nq{q}-after{a}-{'-'.join(f'{k}{v}' for k, v in o.items())}" for _, q, a, o in ATTN_SHAPES])
def test_prompt_attention_workgroup_shapes(name, nq, n_after, over):
    c = build_case(name, **over)
    c.cache.seq_lens[: c.sp.batch // 2] -= np.arange(c.sp.batch // 2, dtype=np.int32) % 40        # ragged, some shorter than n_q
    L = layer_for(c); L.upload(c.cache)
    q32 = _multi_q(c, nq, seed=31)
    got = _prefill_attn(L, c, q32, nq, n_after, int(c.cache.seq_lens.max()))
    ref = O.causal_attn_reconstructed(c.cache, q32.astype(np.float64), c.BK.astype(np.float64), c.BV.astype(np.float64), c.sm_scale,
                                      n_after=n_after)
    check_out(got, ref, "i8", f"prompt attention {name} nq={nq} n_after={n_after} {over}")
    L.close()


@pytest.mark.parametrize("lead", [13.0, 15.5, 19.0])
@pytest.mark.parametrize("where", ["first", "late"])
def test_prompt_attention_many_small_weights(lead, where):
    """One key leads all others by 2^lead: the others' weights are small or subnormal in fp16 where the reference of the
    exponentials is that key's score ("first"), and the wave has to move its reference where the key comes late.  The sum
    of 1990 such weights is up to a fifth of the total and must not be lost."""
    c = build_case("c3_small", batch=2, n_q_heads=2, n_kv_heads=2, context=2000)
    sp = c.sp
    rng = np.random.default_rng(3)
    q32 = np.repeat(_multi_q(c, 1, seed=4), 10, axis=2)                         # ten equal tokens
    t = 5 if where == "first" else 1500
    for b in range(sp.batch):
        k = np.zeros((sp.n_kv_heads, 2000, sp.rank))
        qt = np.einsum("hd,hrd->hr", q32[b, :, 0, 0].astype(np.float64), c.BK.astype(np.float64))
        k[:, t] = qt * (lead * np.log(2.0) / c.sm_scale / (qt * qt).sum(-1))[:, None]
        c.cache.store_rows("k", b, 0, k)
        c.cache.store_rows("v", b, 0, rng.standard_normal((sp.n_kv_heads, 2000, sp.rank)) + 1.0)
        c.cache.seq_lens[b] = 2000
    L = layer_for(c); L.upload(c.cache)
    got = _prefill_attn(L, c, q32, 10, 0, 2000)
    ref = O.causal_attn_reconstructed(c.cache, q32.astype(np.float64), c.BK.astype(np.float64), c.BV.astype(np.float64), c.sm_scale)
    # fp16 weights: 2^-12 relative each, a subnormal one 2^-25 absolute (2^-25 / 2^-19 = 1.6 % of each of the smallest, signs
    # at random over 2000 keys whose sum is 2^-8 of the total); fp16 values 2^-12: 1e-3 covers both
    assert np.linalg.norm(got - ref) <= 1e-3 * np.linalg.norm(ref), np.linalg.norm(got - ref) / np.linalg.norm(ref)
    L.close()


@pytest.mark.parametrize("rank,nq,batch", [(32, 64, 1), (64, 64, 1), (32, 130, 12)])
def test_prompt_attention_denominator_in_fp32(rank, nq, batch):
    """One key of every 32 has the largest score and the only value that is not zero, all others one smaller score: they enter
    through the sum of the weights alone, which has to be taken before the weights are rounded to fp16 (2^-12 relative, the
    same for all of them, times their share of the sum of up to 0.9).  The leading weight is 1 and the value's code times
    its scale is exact."""
    c = build_case("c3_small", batch=batch, n_q_heads=4, n_kv_heads=4, context=512, rank=rank)
    sp = c.sp
    q32 = np.repeat(_multi_q(c, 1, seed=4), nq, axis=2)
    q32 *= np.linspace(1.0, 2.5, nq, dtype=np.float32)[None, None, :, None, None]
    q32 = WI.bf16_exact(q32)
    for b in range(sp.batch):
        k = np.zeros((sp.n_kv_heads, 512, sp.rank))
        qt = np.einsum("hd,hrd->hr", q32[b, :, 0, 0].astype(np.float64), c.BK.astype(np.float64))
        k[:, ::32] = (qt * (1.3 * np.log(2.0) / c.sm_scale / (qt * qt).sum(-1))[:, None])[:, None]
        v = np.zeros((sp.n_kv_heads, 512, sp.rank))
        v[:, ::32] = (np.arange(sp.rank) * 7 % 255 - 127.0) / 16.0              # scale 2^-4, every code an integer
        c.cache.store_rows("k", b, 0, k)
        c.cache.store_rows("v", b, 0, v)
        c.cache.seq_lens[b] = 512
    L = layer_for(c); L.upload(c.cache)
    got = _prefill_attn(L, c, q32, nq, 0, 512)
    ref = O.causal_attn_reconstructed(c.cache, q32.astype(np.float64), c.BK.astype(np.float64), c.BV.astype(np.float64), c.sm_scale)
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    # left: the bf16 pair of U / l (2^-16 per element, signs at random) and the fp32 sums: 2e-5
    assert err.max() <= 4e-5, err.max()
    L.close()


@pytest.mark.parametrize("rank", [32, 64])
def test_prompt_attention_short_prompts_keep_the_waves_busy(rank):
    """64 sequences of 16 tokens, over their own 16 keys, have the query rows of 16 sequences of 64 tokens over 64 keys, and a
    quarter of the scores: with every wave of the launch at work they take about the same time, 1.1 to 1.3 times (waves
    without rows or without a key block to attend to make it 1.8 and 2.6 times)."""
    def us(batch, n):
        desc = W.layer_desc(batch, 32, 32, 128, 4096, rank, 64, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
        ctx = W.wsvd_create(0)
        cb, mb = W.wsvd_cache_bytes(desc)
        g = torch.Generator(device="cuda").manual_seed(1)
        codes = [torch.randint(-127, 128, (cb,), dtype=torch.int8, device="cuda", generator=g) for _ in range(2)]
        meta = [torch.full((mb // 2,), 0.02, dtype=torch.float16, device="cuda") for _ in range(2)]
        lens = torch.full((batch,), n, dtype=torch.int32, device="cuda")
        q = torch.randn(batch, 32, n, 1, 128, device="cuda", generator=g).to(torch.bfloat16)
        B = [(torch.randn(32, rank, 128, device="cuda", generator=g) * rank ** -0.5).to(torch.bfloat16) for _ in range(2)]
        out = torch.zeros(batch, 32, n, 1, 128, device="cuda")
        cache = W.make_cache(*codes, *meta, lens)
        stream = torch.cuda.Stream()
        run = lambda: W.wsvd_prefill_attn(ctx, desc, q, n, 0, *B, cache, n, out, stream)
        torch.cuda.synchronize()
        run()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(20):
                run()
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record(); graph.replay(); b.record(); torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        assert W.wsvd_check(ctx) == 0
        W.wsvd_destroy(ctx)
        return best

    t16, t64 = us(64, 16), us(16, 64)
    assert t16 <= 1.55 * t64, (t16, t64)


@pytest.mark.parametrize("shape", [2, 5, 11, 12, 22, 25])
@pytest.mark.parametrize("batch,n_tok,kv_heads", [(1, 1, 1), (1, 33, 4), (7, 5, 8), (130, 3, 1), (3, 300, 16)])
def test_projection_advances_the_lengths(shape, batch, n_tok, kv_heads):
    """The last workgroup of the tile kernels to count itself advances the lengths: launches of fewer workgroups than counters, of
    many, more sequences than lanes, a sequence that has no room and one that is full; three calls in a row."""
    t_cap = (3 * n_tok + 63) // 64 * 64 + 64
    desc = W.layer_desc(batch, kv_heads, kv_heads, 128, 128, 32, t_cap, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
    ctx = W.wsvd_create(0)
    W.wsvd_ctx_set_option(ctx, "project_shape", shape)
    W.wsvd_ctx_set_option(ctx, "prefill_tiled", 1)
    cb, mb = W.wsvd_cache_bytes(desc)
    codes, meta = [torch.zeros(cb, dtype=torch.uint8, device="cuda") for _ in range(2)], [torch.zeros(mb, dtype=torch.uint8, device="cuda") for _ in range(2)]
    lens = torch.arange(batch, dtype=torch.int32, device="cuda") % 5
    lens[-1] = t_cap - 2 * n_tok if batch == 1 else t_cap          # (alone: full after two calls)
    want = lens.cpu()
    cache = W.make_cache(*codes, *meta, lens)
    x = torch.randn(batch, n_tok, 128, device="cuda").to(torch.bfloat16)
    A = [torch.zeros(W.wsvd_factor_a_bytes(desc), dtype=torch.uint8, device="cuda") for _ in range(2)]
    for call in range(3):
        W.wsvd_prefill_append(ctx, desc, x, None, n_tok, -1, *A, cache)
        full = bool((want + n_tok > t_cap).any())
        want = torch.clamp(want + n_tok, max=t_cap)
        assert W.wsvd_check(ctx) == (W.E_CAPACITY if full else 0), call
        assert (lens.cpu() == want).all(), call
    W.wsvd_destroy(ctx)


def test_new_context_is_ready_on_any_stream():
    """wsvd_create clears the context's counters on the default stream; the projection that counts on them may be the very next
    call, on a stream that does not wait for that one, with the default stream still busy.  The memory is that of contexts before."""
    desc = W.layer_desc(3, 8, 8, 128, 128, 32, 128, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
    cb, mb = W.wsvd_cache_bytes(desc)
    codes, meta = [torch.zeros(cb, dtype=torch.uint8, device="cuda") for _ in range(2)], [torch.zeros(mb, dtype=torch.uint8, device="cuda") for _ in range(2)]
    x = torch.randn(3, 33, 128, device="cuda").to(torch.bfloat16)
    A = [torch.zeros(W.wsvd_factor_a_bytes(desc), dtype=torch.uint8, device="cuda") for _ in range(2)]
    busy = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    for shape in (5, 11, 2, 25):
        lens = torch.zeros(3, dtype=torch.int32, device="cuda")
        cache = W.make_cache(*codes, *meta, lens)
        torch.cuda.synchronize()
        for _ in range(8):
            busy = busy @ busy * 1e-3
        ctx = W.wsvd_create(0)
        W.wsvd_ctx_set_option(ctx, "project_shape", shape)
        W.wsvd_ctx_set_option(ctx, "prefill_tiled", 1)
        for _ in range(3):
            W.wsvd_prefill_append(ctx, desc, x, None, 33, -1, *A, cache, stream=side.cuda_stream)
        assert W.wsvd_check(ctx, stream=side.cuda_stream) == 0
        side.synchronize()
        torch.cuda.synchronize()
        assert (lens.cpu() == 99).all(), shape
        W.wsvd_destroy(ctx)


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("batch,kv_heads,n,past", [(1, 2, 32, 40), (1, 2, 33, 200), (32, 32, 32, 170), (8, 32, 64, 200), (16, 32, 128, 60), (40, 32, 64, 50), (3, 8, 70, 1000)])
def test_prompt_attention_over_infinite_scales(rank, batch, kv_heads, n, past):
    """Scales are the caller's (wsvd_cache_import): the first 40 keys' are infinite and their scores -inf, the first block's for every
    query.  Such keys have weight 0, as masked ones do, whatever the workgroup's shape; everything behind them counts in full."""
    t, dead = past + n, 40
    desc = W.layer_desc(batch, kv_heads, kv_heads, 128, 64, rank, (t + 63) // 64 * 64, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
    ctx = W.wsvd_create(0)
    cb, mb = W.wsvd_cache_bytes(desc)
    planes, meta = [torch.zeros(cb, dtype=torch.uint8, device="cuda") for _ in range(2)], [torch.zeros(mb, dtype=torch.uint8, device="cuda") for _ in range(2)]
    lens = torch.full((batch,), t, dtype=torch.int32, device="cuda")
    cache = W.make_cache(*planes, *meta, lens)
    g = torch.Generator(device="cuda").manual_seed(rank + t)
    kc, vc = (torch.randint(-127, 128, (batch, kv_heads, t, rank), device="cuda", generator=g, dtype=torch.int8) for _ in range(2))
    kc[:, :, :dead] = torch.randint(-127, 0, (batch, kv_heads, dead, rank), device="cuda", generator=g, dtype=torch.int8)
    ks, vs = (0.001 * (1 + torch.rand(batch, kv_heads, t, device="cuda", generator=g)) for _ in range(2))
    ks[:, :, :dead] = float("inf")
    ks, vs = ks.half(), vs.half()
    W.wsvd_cache_import(ctx, desc, 0, kc, ks, 0, t, cache)
    W.wsvd_cache_import(ctx, desc, 1, vc, vs, 0, t, cache)
    q = torch.randn(batch, kv_heads, n, 128, device="cuda", generator=g).abs().to(torch.bfloat16)
    BK, BV = (torch.randn(kv_heads, rank, 128, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    BK = BK.abs()
    out = torch.full((batch, kv_heads, n, 1, 128), float("nan"), device="cuda")
    W.wsvd_prefill_attn(ctx, desc, q, n, 0, BK, BV, cache, t, out)
    assert W.wsvd_check(ctx) == 0
    C, V = kc.double()[:, :, dead:] * ks.double()[:, :, dead:, None], vc.double()[:, :, dead:] * vs.double()[:, :, dead:, None]
    s = (q.double() @ BK.double().transpose(1, 2)) @ C.transpose(2, 3) / 128 ** 0.5
    late = torch.arange(t - dead, device="cuda")[None, :] + dead > torch.arange(n, device="cuda")[:, None] + past
    ref = (torch.softmax(s.masked_fill(late, float("-inf")), -1) @ V) @ BV.double()
    err = (out[:, :, :, 0].double() - ref).norm() / ref.norm()
    assert err <= 2e-3, float(err)                               # (fp16 weights: 2^-12 each, seen 2e-4 with finite scales)
    W.wsvd_destroy(ctx)

"""Rotary decode attention: the form with a rotation table (more (sequence, kv head) units than CUs, one query head, rank 32)
at the edges of its tiles and runs of two tiles, and the split of few units over several workgroups, against the oracle; the
number of workgroups that is chosen against the others that can be asked for."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2604_02570_amd as W
from cases import build_case
from harness import as_dtype_dev, q_to_device
from test_gpu_parity import check_out, layer_for

pytestmark = pytest.mark.gpu


def _rope(name, base, options=(), **over):
    c = build_case(name, **over)
    L = layer_for(c); L.upload(c.cache)
    for option, value in options:
        W.wsvd_ctx_set_option(L.ctx, option, value)
    qd, qs, q64 = q_to_device(c.q32[0], c.sp.q_dtype)
    BKd, BVd = as_dtype_dev(c.BK, "bf16"), as_dtype_dev(c.BV, "bf16")
    got = L.attend_rope(qd, qs, BKd, BVd, int(c.cache.seq_lens.max()), base)
    again = L.attend_rope(qd, qs, BKd, BVd, int(c.cache.seq_lens.max()), base)
    assert (got == again).all()
    ref = O.decode_attn_rope_reconstructed(c.cache, q64, c.BK.astype(np.float64), c.BV.astype(np.float64), c.sm_scale, base)
    check_out(got, ref, "rope", f"rope {name} {over}")
    L.close()


# 288 units: one to four waves with a tile, a last run of one tile, several runs per wave; every length from 1 on in a ragged batch
@pytest.mark.parametrize("over", [dict(context=1), dict(context=64), dict(context=65), dict(context=130), dict(context=300), dict(context=513),
                                  dict(context=577, d_head=64), dict(context=700, ragged=(1, 700))],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()))
@pytest.mark.parametrize("name", ["c3_small", "c4_small"])
def test_rope_table(name, over):
    _rope(name, 10000.0, **{**dict(batch=9, n_q_heads=32, n_kv_heads=32, ragged=()), **over})


# the same split over two to nine workgroups, which has to be asked for: chunks of one run for every wave and of single tiles, a
# chunk's last run of one tile, a last chunk of few rows, sequences that end before the later chunks begin
@pytest.mark.parametrize("min_chunk,over", [(512, dict(context=1024)), (576, dict(context=1100)), (256, dict(context=2050)), (1024, dict(context=2049, d_head=64)),
                                            (320, dict(context=1300, ragged=(1, 1300)))], ids=["512", "576", "256", "1024-d64", "320-ragged"])
@pytest.mark.parametrize("name", ["c3_small", "c4_small"])
def test_rope_table_split_over_workgroups(name, min_chunk, over):
    _rope(name, 10000.0, options=(("wg_per_cu", 64), ("min_chunk", min_chunk)),
          **{**dict(batch=9, n_q_heads=32, n_kv_heads=32, ragged=()), **over})


@pytest.mark.parametrize("q_dtype", ["f32", "bf16", "i8"])
def test_rope_table_query_types_and_base(q_dtype):
    _rope("c3_small", 500.0, batch=9, n_q_heads=32, n_kv_heads=32, context=260, q_dtype=q_dtype)


# (8 units: one chunk up to 1100 rows, two to eight from 1300 on)
@pytest.mark.parametrize("over", [dict(context=1023), dict(context=1024), dict(context=1100), dict(context=2050, rank=64), dict(context=1500, n_q_heads=8),
                                  dict(context=1300), dict(context=2049, ragged=(3, 2049)), dict(context=4100)],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()))
def test_rope_split_over_workgroups(over):
    _rope("c3_small", 10000.0, **{**dict(batch=2, n_q_heads=4, n_kv_heads=4), **over})


# just above and below the counts of units that divide the CUs
@pytest.mark.parametrize("units,rows", [(86, 1500), (88, 2048), (136, 2048), (136, 8192), (52, 4096), (43, 8192), (288, 1500), (128, 2048), (16, 4096)])
def test_rope_takes_a_fitting_number_of_chunks(units, rows):
    """The chunks of the context that are taken by themselves are about as fast as the best number asked for (one workgroup
    too many is a second round of them: 1.2 to 1.5 times)."""
    hkv = next(h for h in (8, 4, 1) if units % h == 0)
    desc = W.layer_desc(units // hkv, hkv, hkv, 128, 4096, 32, (rows + 63) // 64 * 64, "i8", "bf16", "bf16", "bf16", "f32", 0.0)
    ctx = W.wsvd_create(0)
    ws = torch.empty(W.wsvd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    W.wsvd_set_workspace(ctx, ws)
    cb, mb = W.wsvd_cache_bytes(desc)
    g = torch.Generator(device="cuda").manual_seed(1)
    codes = [torch.randint(-127, 128, (cb,), dtype=torch.int8, device="cuda", generator=g) for _ in range(2)]
    meta = [torch.full((mb // 2,), 0.02, dtype=torch.float16, device="cuda") for _ in range(2)]
    lens = torch.full((units // hkv,), rows, dtype=torch.int32, device="cuda")
    q = torch.randn(units // hkv, hkv, 128, device="cuda", generator=g).to(torch.bfloat16)
    B = [(torch.randn(hkv, 32, 128, device="cuda", generator=g) * 32 ** -0.5).to(torch.bfloat16) for _ in range(2)]
    out = torch.zeros(units // hkv, hkv, 128, device="cuda")
    cache = W.make_cache(*codes, *meta, lens)
    stream = torch.cuda.Stream()
    run = lambda: W.wsvd_decode_attn_rope(ctx, desc, q, None, *B, cache, rows, 10000.0, out, stream)

    def us(wg_per_cu, min_chunk):
        W.wsvd_ctx_set_option(ctx, "wg_per_cu", wg_per_cu)
        W.wsvd_ctx_set_option(ctx, "min_chunk", min_chunk)
        torch.cuda.synchronize()
        run()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(20):
                run()
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record(); graph.replay(); b.record(); torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    t = {k: us(64, ((rows + k - 1) // k + 63) // 64 * 64) for k in (1, 2, 3, 4, 6)}
    t[0] = us(4, 0)
    assert W.wsvd_check(ctx) == 0
    assert t[0] <= 1.12 * min(t.values()), t
    W.wsvd_destroy(ctx)

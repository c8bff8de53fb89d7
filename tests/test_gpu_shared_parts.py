"""Shared-latent decode attention where its launches change shape: value dims over one, two and four workgroups, one and
several chunks per split, sequence counts in and out of whole groups of eight, both merge workgroups, empty sequences
among them.  The oracle computes a sample of (sequence, head) pairs.  And the plan of large batches by their times."""
import numpy as np
import pytest
import torch

import paper_2604_02570_amd as W
from test_gpu_parity import check_out
from test_gpu_shared import H, SharedCase

pytestmark = pytest.mark.gpu

#      rank, d, t_cap, lengths, (splits, parts)                    what a workgroup walks
CASES = [
    (1024, 128, 5120, [4999], (32, 4)),                                      # up to two chunks
    (1024, 64, 1024, [1000 - 61 * b for b in range(17)], (7, 2)),            # up to two
    (1024, 128, 2048, [(2048 * (b % 5)) // 4 for b in range(24)], (10, 1)),  # up to two, all registers, empty sequences
    (1024, 128, 2048, [(2048 * (b % 5)) // 4 for b in range(20)], (6, 2)),   # up to three, empty sequences
    (512, 128, 1024, [1023, 1], (8, 4)),                                     # one
    (512, 64, 1280, [1280 - 100 * b for b in range(9)], (10, 2)),            # one
    (512, 128, 640, [640 - 16 * b for b in range(40)], (5, 1)),              # one
    (512, 128, 896, [896 - 22 * b for b in range(40)], (6, 1)),              # up to two
    (256, 128, 512, [129, 0, 512], (4, 2)),                                  # one
    (3712, 128, 1280, [1280 - 97 * b for b in range(12)], (10, 2)),          # two workgroups for four slabs of value dims, one
    (256, 64, 1024, [1024 - 31 * b for b in range(33)], (7, 1)),             # up to two
    (1024, 128, 768, [768 - 11 * b for b in range(66)], (3, 1)),             # up to two
    (1024, 64, 384, [384 - 2 * b for b in range(130)], (1, 1)),              # up to three
    (256, 128, 512, [512 - 3 * b for b in range(130)], (2, 1)),              # up to two, two workgroups to a CU
]


@pytest.mark.parametrize("rank,d,t_cap,lens,plan", CASES, ids=[f"r{c[0]}-d{c[1]}-b{len(c[3])}" for c in CASES])
def test_shared_latent_launch_shapes(rank, d, t_cap, lens, plan):
    assert W.wsvd_test_shared_plan(len(lens), rank, t_cap) == plan
    print(f"shared latent: rank {rank}, d {d}, {len(lens)} sequences, t_cap {t_cap}", flush=True)
    c = SharedCase(len(lens), rank, d, lens, t_cap)
    ctx = W.wsvd_create(0)
    got = c.run(ctx)
    W.wsvd_destroy(ctx)
    for b, n in enumerate(lens):
        if n == 0:
            assert (got[b] == 0).all()
    assert np.isfinite(got).all()
    rng = np.random.default_rng(rank + len(lens))
    pairs = [(b, int(rng.integers(0, H))) for b in sorted({0, len(lens) - 1, *(int(x) for x in rng.integers(0, len(lens), 6))}) if lens[b]]
    check_out(got, c.oracle(heads=pairs), "i8", f"shared latent rank {rank}, {len(lens)} sequences, {len(pairs)} sampled pairs")


def _us(batch, rows, rank):
    """us per call of `batch` sequences of `rows` rows (a graph of ten calls)."""
    d, t_cap = 128, (rows + 127) // 128 * 128
    ctx = W.wsvd_create(0)
    g = torch.Generator(device="cuda").manual_seed(1)
    codes = [torch.randint(-127, 128, (batch, t_cap * rank), dtype=torch.int8, device="cuda", generator=g) for _ in range(2)]
    scale = torch.full((batch, t_cap), 0.02, dtype=torch.float16, device="cuda")
    q = torch.randn(batch, H, d, device="cuda", generator=g).to(torch.bfloat16)
    B = [(torch.randn(H, rank, d, device="cuda", generator=g) * rank ** -0.5).to(torch.bfloat16) for _ in range(2)]
    lens = torch.full((batch,), rows, dtype=torch.int32, device="cuda")
    ws = torch.empty(W.wsvd_shared_workspace_bytes(batch, H, d, rank, t_cap), dtype=torch.uint8, device="cuda")
    out = torch.zeros(batch, H, d, device="cuda")
    stream = torch.cuda.Stream()
    run = lambda: W.wsvd_decode_attn_shared(ctx, batch, H, d, rank, t_cap, 0.0, q, *B, *codes, scale, scale, lens, ws, out, stream)
    torch.cuda.synchronize()
    run()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for _ in range(10):
            run()
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record(); graph.replay(); b.record(); torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    assert W.wsvd_check(ctx) == 0
    W.wsvd_destroy(ctx)
    return best


# one sequence more than a count that divides the CUs, and full batches against a quarter of them, which has the same plan but
# for the splits: 1.19, 1.25 and 2.7 times (half as many workgroups as CUs, or the scores computed twice: 1.45, 1.43 and 3.8)
@pytest.mark.parametrize("rank,rows,few,many,limit", [(1024, 2048, 64, 65, 1.33), (256, 2048, 128, 129, 1.35), (1024, 8192, 16, 64, 3.2)])
def test_shared_latent_large_batches_keep_the_cus_busy(rank, rows, few, many, limit):
    t_few, t_many = _us(few, rows, rank), _us(many, rows, rank)
    assert t_many <= limit * t_few, (t_few, t_many)

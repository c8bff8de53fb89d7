"""Shared-latent decode attention where its launches change shape: value dims over one, two and four workgroups, one and
several chunks per split, sequence counts in and out of whole groups of eight, both merge workgroups, empty sequences
among them.  The oracle computes a sample of (sequence, head) pairs."""
import numpy as np
import pytest

import paper_2604_02570_amd as W
from test_gpu_parity import check_out
from test_gpu_shared import H, SharedCase

pytestmark = pytest.mark.gpu

#      rank, d, t_cap, lengths                                      parts, chunks per split
CASES = [
    (1024, 128, 5120, [4999]),                                     # 4, two
    (1024, 64, 1024, [1000 - 61 * b for b in range(17)]),          # 2, up to two
    (1024, 128, 2048, [(2048 * (b % 5)) // 4 for b in range(24)]),   # 2, up to four, empty sequences
    (512, 128, 1024, [1023, 1]),                                   # 4, one
    (512, 64, 1280, [1280 - 100 * b for b in range(9)]),           # 2, one
    (512, 128, 640, [640 - 16 * b for b in range(40)]),            # 1, one
    (256, 128, 512, [129, 0, 512]),                                # 2, one
    (3712, 128, 1280, [1280 - 97 * b for b in range(12)]),         # two workgroups for four slabs of value dims, one
    (256, 64, 1024, [1024 - 31 * b for b in range(33)]),           # 1, two
]


@pytest.mark.parametrize("rank,d,t_cap,lens", CASES, ids=[f"r{c[0]}-d{c[1]}-b{len(c[3])}" for c in CASES])
def test_shared_latent_launch_shapes(rank, d, t_cap, lens):
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

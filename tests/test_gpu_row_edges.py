"""Edges of the row kernels' pass counts, of the latent store's look-ahead and of the append's walk over the hidden states:
the oracle comparisons of the neighbouring files at the sizes where a wrong count would show."""
import numpy as np
import pytest
import torch

import paper_2604_02570_amd as W

import test_gpu_block as TB
import test_gpu_layer as TL
import test_gpu_parity as TP

pytestmark = pytest.mark.gpu

# 1024 threads x 4 channels a pass (16 bytes of the row each): one element on either side of every pass boundary
EDGES = [4092, 4096, 4100, 8192, 8196, 12288, 12292]


@pytest.mark.parametrize("cols", EDGES)
def test_rmsnorm_and_swiglu_pass_edges(cols):
    TL.test_rmsnorm_quant_matches_oracle(2, cols, cols % 8 == 0)
    TL.test_rmsnorm_quant_matches_oracle(3, cols, cols % 8 != 0)
    TL.test_swiglu_quant_matches_oracle(2, cols)


@pytest.mark.parametrize("cols,dt", [(c, "f32") for c in EDGES] + [(c, "bf16") for c in (8184, 8192, 8200, 16384, 16392)])
def test_quantize_act_pass_edges(cols, dt):
    TP.test_quantize_act_i8_bit_exact(3, cols, dt)


# 2 Hkv r latents per sequence over 1024 threads, four of them requested ahead: below, at and past that count
@pytest.mark.parametrize("hkv,r", [(1, 32), (16, 32), (17, 32), (32, 64), (33, 64)])
def test_latent_store_look_ahead_edges(hkv, r):
    TB.test_latent_store_matches_oracle("c3_small", dict(n_q_heads=hkv, n_kv_heads=hkv, rank=r, batch=3, context=70))


# (batch, d_model): shares of the hidden states with fewer and more 16-byte pieces per row than threads, walks that do and
# do not divide the workgroup, both group sizes and a partly filled last group
@pytest.mark.parametrize("batch,d_model", [(1, 64), (5, 192), (17, 1088), (33, 3584), (16, 4160), (9, 16448)])
@pytest.mark.parametrize("name,rank", [("c3_small", 32), ("c3_small", 64), ("c4_small", 32), ("c2_small", 32)])
def test_append_walk_edges(name, rank, batch, d_model):
    TP.test_append_matches_oracle(name, dict(rank=rank, n_q_heads=2, n_kv_heads=2, batch=batch, d_model=d_model, context=40))


@pytest.mark.parametrize("scale", [2.0 ** -24, 5 * 2.0 ** -24, 0.0123, 0.1, 1.0, 3.1, 1023.5, 65504.0])
def test_codes_at_rounding_boundaries(scale):
    """Values (k + 1/2) s and their fp32 neighbours in a row whose scale is the fp16 number s, and one infinite row: the
    quantiser's quotients have to be those of the division, bit for bit."""
    s = np.float32(np.float16(scale))
    half = ((np.arange(-127, 127) + 0.5) * np.float64(s)).astype(np.float32)
    row = np.concatenate([half, np.nextafter(half, np.float32(np.inf)), np.nextafter(half, np.float32(-np.inf)), np.float32([127 * s] * 6)])
    rng = np.random.default_rng(5)
    x = np.stack([row, rng.permutation(row), np.where(np.arange(row.size) == 7, np.float32(np.inf), row), -row])
    c = np.empty(x.shape, np.int8)
    sc = np.empty(len(x), np.float16)
    with np.errstate(invalid="ignore", over="ignore"):
        for i, r in enumerate(x):
            a = np.float32(np.abs(r).max()) / np.float32(127)
            sc[i] = np.float16(min(max(a, np.float32(2.0 ** -24)), np.float32(65504.0)))
            c[i] = np.clip(np.rint(r / np.float32(sc[i])), -127, 127)
    ctx = W.wsvd_create(0)
    codes = torch.zeros(x.shape, dtype=torch.int8, device="cuda"); scales = torch.zeros(len(x), dtype=torch.int16, device="cuda")
    W.wsvd_quantize_act_i8(ctx, torch.from_numpy(x).cuda(), "f32", *x.shape, codes, scales)
    assert (scales.cpu().numpy().view(np.float16) == sc).all()
    assert (codes.cpu().numpy() == c).all()
    W.wsvd_destroy(ctx)

"""Rotary decode attention: the form with a rotation table (more (sequence, kv head) units than CUs, one query head, rank 32)
at the edges of its tiles and runs of two tiles, and the split of few units over several workgroups, against the oracle."""
import numpy as np
import pytest

import oracle as O
from cases import build_case
from harness import as_dtype_dev, q_to_device
from test_gpu_parity import check_out, layer_for

pytestmark = pytest.mark.gpu


def _rope(name, base, **over):
    c = build_case(name, **over)
    L = layer_for(c); L.upload(c.cache)
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


@pytest.mark.parametrize("q_dtype", ["f32", "bf16", "i8"])
def test_rope_table_query_types_and_base(q_dtype):
    _rope("c3_small", 500.0, batch=9, n_q_heads=32, n_kv_heads=32, context=260, q_dtype=q_dtype)


@pytest.mark.parametrize("over", [dict(context=1023), dict(context=1024), dict(context=1100), dict(context=2050, rank=64), dict(context=1500, n_q_heads=8)],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()))
def test_rope_split_over_workgroups(over):
    _rope("c3_small", 10000.0, **{**dict(batch=2, n_q_heads=4, n_kv_heads=4), **over})

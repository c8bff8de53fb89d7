"""Prompt projection: every kernel shape of the dispatch stores the rows the oracle's projection gives, for sizes at the
edges of its token tiles (one tile, one more, one less, several with a remainder) and sequences that already hold rows."""
import numpy as np
import pytest

import paper_2604_02570_amd as W
import wsvd_inputs as WI
from cases import build_case
from harness import as_dtype_dev, check_i8_rows
from test_gpu_parity import layer_for
from test_gpu_prefill import _check_i4_rows, _latents64

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

"""CPU-side checks of the boundary: the shared library loads and exports every symbol include/wsvd.h
declares, the binding mirrors them, and host-only calls validate their arguments (no kernel is launched)."""
import ctypes
import os
import re
import struct
import subprocess
import tempfile

import pytest

import paper_2604_02570_amd as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    """Every function include/*.h declares: the product boundary (wsvd.h) and the test / profiling hooks (wsvd_test.h)."""
    names = set()
    for header in ("wsvd.h", "wsvd_test.h"):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(wsvd_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_header_symbols_exported_and_bound():
    names = declared_functions()
    assert "wsvd_latent_append" in names and "wsvd_decode_attn" in names and len(names) >= 14
    lib = W.lib()
    for n in names:
        assert hasattr(lib, n), f"libwsvd.so does not export {n}"
        assert hasattr(W, n) or n == "wsvd_status_str", f"python binding lacks {n}"
    assert sorted(W.EXPORTS) == names


def test_status_strings():
    for code in range(9):
        assert W.status_str(code) != "unknown status"
    assert W.status_str(99) == "unknown status"


def test_struct_sizes_match_header():
    assert ctypes.sizeof(W.LayerDesc) == 13 * 4
    assert ctypes.sizeof(W.Cache) == 5 * ctypes.sizeof(ctypes.c_void_p)


def test_host_only_validation_and_sizes():
    d = W.layer_desc(16, 32, 32, 128, 4096, 32, 2048, "i8", "bf16", "bf16", "i8")
    codes, meta = W.wsvd_cache_bytes(d)
    assert codes == 16 * 32 * 2048 * 32 and meta == 16 * 32 * 2048 * 2
    assert 2 * (codes + meta) == 71303168          # bytes one attention call streams at this shape
    d4 = W.layer_desc(64, 32, 32, 128, 4096, 32, 4160, "i4", "bf16", "bf16", "i8")
    codes, meta = W.wsvd_cache_bytes(d4)
    assert codes == 64 * 32 * 4160 * 16 and meta == 64 * 32 * 4160 * 4
    assert W.wsvd_workspace_bytes(d) >= 65536
    for kw, status in ((dict(d_head=96), 2), (dict(rank=48), 2), (dict(n_q_heads=33), 2), (dict(t_cap=100), 2),
                       (dict(latent_dtype="i4", rank=64), 6), (dict(factor_dtype="f32"), 3), (dict(out_dtype="i8"), 3)):
        args = dict(batch=16, n_q_heads=32, n_kv_heads=32, d_head=128, d_model=4096, rank=32, t_cap=2048, latent_dtype="i8",
                    factor_dtype="bf16", x_dtype="bf16", q_dtype="i8", out_dtype="f32")
        args.update(kw)
        with pytest.raises(W.WsvdError) as e:
            W.wsvd_cache_bytes(W.layer_desc(**args))
        assert e.value.status == status, kw
    with pytest.raises(W.WsvdError) as e:
        W.wsvd_ctx_set_option(None, "max_threads", 256)        # a context is required: the setting lives in it
    assert e.value.status == W.E_NULL


def test_shared_latent_plan_fits_its_workspace():
    """For every batch the workspace holds the query images and the partial results of the splits that are launched, no
    workgroup above rank 1024 gets more than four chunks of 128 tokens, and up to there a round of workgroups is not exceeded
    (two to a CU at rank 256)."""
    for rank in (256, 512, 1024, 1152, 2560, 4096):
        for t_cap in (128, 512, 2048, 8192, 16384):
            for batch in (*range(1, 70), 85, 86, 127, 128, 129, 200, 255, 256, 257, 600):
                splits, parts = W.wsvd_test_shared_plan(batch, rank, t_cap)
                chunks = t_cap // 128
                need = 4 * batch * 32 * (rank + splits * (rank + 2))
                assert need <= W.wsvd_shared_workspace_bytes(batch, 32, 128, rank, t_cap), (rank, t_cap, batch)
                assert 1 <= splits <= min(32, chunks) and parts in ((1, 2, 3, 4) if rank > 1024 else (1, 2, 4)), (rank, t_cap, batch)
                if rank > 1024:
                    assert -(-chunks // splits) <= 4, (rank, t_cap, batch)
                else:
                    assert batch * splits * parts <= max(512 if rank == 256 else 256, batch), (rank, t_cap, batch)


def kernel_scratch_bytes():
    """Scratch memory per lane of every kernel of the built library, by (mangled) name: the notes of its gfx950 code objects."""
    data = open(W.LIB_PATH, "rb").read()
    magic, sizes = b"__CLANG_OFFLOAD_BUNDLE__", {}
    for m in re.finditer(magic, data):
        (n,) = struct.unpack_from("<Q", data, m.start() + len(magic))
        at = m.start() + len(magic) + 8
        for _ in range(n):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            at += 24
            target, at = data[at:at + name], at + name
            if size == 0 or b"gfx950" not in target:
                continue
            with tempfile.NamedTemporaryFile(suffix=".co") as f:
                f.write(data[m.start() + offset:m.start() + offset + size]); f.flush()
                notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", f.name], capture_output=True, text=True, check=True).stdout
            for kernel in notes.split("\n  - ")[1:]:
                name = re.search(r"\.name:\s+(_Z\S+)", kernel)
                if name:
                    sizes[name[1]] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel)[1])
    return sizes


def test_row_and_prompt_kernels_use_no_scratch_memory():
    """The kernels of the append, the latent store, the row quantisers and the prompt keep everything in registers (the
    prompt projection without LDS, for sequences of 2^31 bytes and more and for rank 128, is the known exception)."""
    sizes = kernel_scratch_bytes()
    for part, least in (("k_latent_store", 3), ("k_append", 6), ("k_prefill_attn", 24), ("k_prefill_project_direct", 6),
                        ("k_prefill_project_lds", 3), ("k_shared", 14), ("k_rmsnorm_quant", 8), ("k_swiglu_quant", 4), ("k_quantize_act", 9), ("k_attn_generic", 96)):
        found = {k: v for k, v in sizes.items() if part in k}
        assert len(found) >= least, (part, sorted(found))
        assert not any(found.values()), {k: v for k, v in found.items() if v}

"""CPU-only: the C-ABI library loads and exports every entry point include/ht.h declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2404_12022_amd", "libht.so")


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "ht.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ht_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_four_named_entry_points():
    names = declared_symbols()
    for must in ("ht_init_model", "ht_transfer", "ht_tree_verify_step", "ht_accept_and_compact"):
        assert must in names


def test_library_exports_every_declared_symbol():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    lib = ctypes.CDLL(LIB)
    for name in declared_symbols():
        assert hasattr(lib, name), f"{name} is declared in ht.h but not exported by libht.so"


def test_binding_names_match_the_header():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    import paper_2404_12022_amd.binding as B
    assert sorted(B.EXPORTS) == declared_symbols()
    # host-only argument checks: no GPU is touched before validation fails
    cfg = B.ht_config()
    out = ctypes.c_size_t(0)
    assert B.lib.ht_workspace_bytes(ctypes.byref(cfg), ctypes.byref(out)) == B.HT_EINVAL
    assert b"dimension" in B.lib.ht_last_error()
    assert B.lib.ht_padded_rows(1) == 16 and B.lib.ht_padded_rows(64) == 64 and B.lib.ht_padded_rows(65) == 128
    from ht_inputs import WORKLOADS
    good = B.make_config(WORKLOADS["llama7b"])
    assert B.ht_workspace_bytes(good) > 32 * 2 * 1024 * 4096 * 2          # at least the KV cache
    good.transfer_layer[1] = 25                                            # 24, 25, 24: layers may not decrease
    assert B.lib.ht_workspace_bytes(ctypes.byref(good), ctypes.byref(out)) == B.HT_EINVAL
    good.transfer_layer[2] = 30                                            # 24, 25, 30 is fine
    assert B.lib.ht_workspace_bytes(ctypes.byref(good), ctypes.byref(out)) == B.HT_OK


def test_binding_constants_match_the_header():
    """Limits and codes the binding re-types (it cannot include a C header) against include/ht.h."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    import paper_2404_12022_amd.binding as B
    text = open(os.path.join(ROOT, "include", "ht.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    enums = dict((k, int(v)) for k, v in re.findall(r"\b(HT_[A-Z_0-9]+)\s*=\s*(-?\d+)", text))
    for name in ("HT_OK", "HT_EINVAL", "HT_ECAPACITY", "HT_ETREE", "HT_ESTATE", "HT_EHIP", "HT_EUNSUPPORTED", "HT_F32", "HT_BF16",
                 "HT_MAX_TRANSFER", "HT_MAX_TREE", "HT_MAX_ROWS", "HT_MAX_TOPK", "HT_MAX_LOOP_STEPS", "HT_BUF_DRAFT_LOGITS",
                 "HT_BUF_K_CACHE", "HT_BUF_V_CACHE", "HT_BUF_FUSED_DRAFT_LOGITS", "HT_BUF_TREE_PARENT", "HT_BUF_TREE_RANK"):
        assert getattr(B, name) == enums[name], name
    m = re.search(r"#define\s+HT_NOALLOC_SCRATCH_BYTES\s+\((\d+)u\s*<<\s*(\d+)\)", text)
    assert B.HT_NOALLOC_SCRATCH_BYTES == int(m.group(1)) << int(m.group(2))
    assert B.lib.ht_padded_rows(129) == 256 and B.lib.ht_padded_rows(256) == 256


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_torch_internals(monkeypatch, missing):
    """A torch build without the short way to the current stream's handle: the long one."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    import types
    import torch
    import paper_2404_12022_amd.binding as B
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 40 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 2, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=7))
    assert B._stream_ptr() == 42
    monkeypatch.delattr(torch._C, missing)
    assert B._stream_ptr() == 7 and B._stream_ptr(types.SimpleNamespace(cuda_stream=9)) == 9


def test_the_tile_that_a_product_takes():
    """The rule that picks the tile of a product of more than 128 rows, at the shapes its comment names (M, N, K, splits): 0 to 7
    256 x 256, 128 x 256, 192 x 256, 192 x 128, 128 x 128, 96 x 128, 64 x 128, 64 x 64; 8 whole rounds and the rest."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    import ctypes as C
    import paper_2404_12022_amd.binding as B
    tile = getattr(B.lib, "_ZN2ht12gemm_tile_ofEiiii")
    tile.restype, tile.argtypes = C.c_int, [C.c_int] * 4
    for shape, want in {(384, 1024, 1024, 1): 7, (256, 4096, 4096, 2): 6, (160, 12288, 4096, 1): 5, (256, 12288, 4096, 1): 5,
                        (256, 4096, 11008, 4): 4, (256, 22016, 4096, 1): 3, (512, 12288, 4096, 1): 3, (256, 32000, 4096, 1): 1,
                        (512, 22016, 4096, 1): 2, (1024, 12288, 4096, 1): 2, (512, 27648, 5120, 1): 0, (4096, 12288, 4096, 1): 0,
                        (2048, 27648, 5120, 1): 8, (1024, 22016, 4096, 1): 8, (1025, 14864, 2048, 1): 3, (1800, 12288, 2048, 1): 8}.items():
        assert tile(*shape) == want, (shape, tile(*shape))


def test_bench_refuses_more_than_one_gpu():
    """One GPU is the whole target: `bench.py --gpus N` with N > 1 exits with a message and prints no result line."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and not r.stdout.strip()


def test_workspace_holds_what_its_model_reads():
    """fp32 models keep no K-split partial sums and no gate | up buffer: what a row of a pass adds to the workspace is the
    residual stream, q, the attention output, the activation, the logits, one saved residual per transfer step and small
    tables.  bf16 models add the activations of a prompt pass once, however long the cache."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    import paper_2404_12022_amd.binding as B
    from ht_inputs import WORKLOADS
    wl = WORKLOADS["llama7b"].with_(n_layers=2, transfer_layers=(1, 1, 1))
    d, qd, f, v, k = wl.d_model, wl.n_heads * wl.head_dim, wl.d_ffn, wl.vocab, wl.k
    f32 = wl.with_(dtype="f32")
    rows = B.ht_workspace_bytes(B.make_config(f32, max_tree=256)) - B.ht_workspace_bytes(B.make_config(f32, max_tree=128))
    live = 4 * (d + 2 * qd + f + v + k * d + wl.head_dim)
    attention = 4 * 16 * wl.n_heads * (wl.head_dim + 2)                  # partial outputs of the key slices
    assert 128 * live <= rows <= 128 * (live + attention + 1024)
    short, long = (B.ht_workspace_bytes(B.make_config(wl, max_cache=c)) for c in (2048, 8192))
    cache = 6144 * 2 * 2 * 2 * wl.n_kv_heads * wl.head_dim               # slots x layers x (K, V) x bytes
    assert cache <= long - short <= cache + 6144 * 16                    # prompt tokens and loss terms beside it

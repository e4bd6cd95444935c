"""Prompts on packed bf16 models: the length picks the kernels (streaming products up to 128 rows, token-tiled above, passes
of equal length past the largest one), the caches, the transfer source and the root must not show it."""
import pytest

import gpu_harness as H
from helpers import prompt_of
from ht_inputs import WORKLOADS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 17, 128, 129, 200, 513])
@pytest.mark.parametrize("heads", ["full", "grouped"])
def test_prompt_of_any_length_fills_the_cache(n, heads):
    wl = WORKLOADS["tiny_t123_bf16"].with_(prompt_len=n, max_cache=(n + 32 + 7) // 8 * 8, seed=n)
    if heads == "grouped":
        wl = wl.with_(n_heads=8, n_kv_heads=2, d_ffn=336)
    print(f"prompt of {n} tokens, {heads} heads", flush=True)
    sc = H.StepCompare(wl, prompt=prompt_of(wl))
    sc.check_prefill()
    sc.step(require_same_tokens=False)


def test_prompt_longer_than_one_pass():
    wl = WORKLOADS["tiny_bf16"].with_(prompt_len=2061, max_cache=2104, n_heads=2, n_kv_heads=1, d_model=128, d_ffn=336)
    print("prompt of two passes", flush=True)
    sc = H.StepCompare(wl, prompt=prompt_of(wl))
    sc.check_prefill()
    sc.step(require_same_tokens=False)


def test_a_second_prompt_replaces_the_first():
    import torch
    import paper_2404_12022_amd.binding as B
    wl = WORKLOADS["tiny_bf16"].with_(prompt_len=300, max_cache=512)
    a, b = prompt_of(wl), prompt_of(wl.with_(prompt_len=150, seed=3))
    gpu = H.gpu_model(wl)
    gpu.ht_prefill(b)
    want = [gpu.ht_get_buffer(w, l)[..., :150].clone() if w == B.HT_BUF_V_CACHE else gpu.ht_get_buffer(w, l)[:150].clone()
            for w in (B.HT_BUF_K_CACHE, B.HT_BUF_V_CACHE) for l in range(wl.n_layers)]
    root = gpu.ht_get_buffer(B.HT_BUF_ROOT).clone()
    gpu.ht_prefill(a)
    gpu.ht_prefill(b)
    got = [gpu.ht_get_buffer(w, l)[..., :150] if w == B.HT_BUF_V_CACHE else gpu.ht_get_buffer(w, l)[:150]
           for w in (B.HT_BUF_K_CACHE, B.HT_BUF_V_CACHE) for l in range(wl.n_layers)]
    assert all(torch.equal(x, y) for x, y in zip(want, got)) and torch.equal(root, gpu.ht_get_buffer(B.HT_BUF_ROOT))
    assert gpu.ht_cache_len() == 150
    gpu.close()


def test_probabilities_of_a_long_causal_range_are_rounded_below_one():
    """64 keys, then keys that score a little higher: relative to the first ones the later probabilities would be 1.0035 and
    lose all of the .0035 in bf16; relative to the running maximum they are 1 and only the first ones (0.9965) are rounded."""
    import ctypes as C
    import torch
    import paper_2404_12022_amd.binding as B

    class Tree(C.Structure):
        _fields_ = [(f, C.c_void_p) for f in ("parent", "depth", "rank", "anc")]

    rows, Hq, Hkv, hd = 600, 2, 1, 128
    cap = (rows + 7) // 8 * 8
    q = torch.zeros(rows, Hq, hd, dtype=torch.bfloat16, device=H.DEV)
    k = torch.zeros(cap, Hkv, hd, dtype=torch.bfloat16, device=H.DEV)
    q[:, :, 0] = 1.0
    k[:64, :, 0] = 1.0
    k[64:, :, 0] = 1.0390625                           # exp(0.0390625 / sqrt(128)) = 1.00346
    v = torch.ones(Hkv, hd, cap, dtype=torch.bfloat16, device=H.DEV)
    v[:, 1] = 2.0
    anc = torch.zeros(256, B.HT_MAX_ROWS // 64, dtype=torch.int64)
    for r in range(256):                               # a chain: row r sees rows 0 .. r
        for w in range(B.HT_MAX_ROWS // 64):
            bits = min(max(r + 1 - 64 * w, 0), 64)
            anc[r, w] = -1 if bits == 64 else (1 << bits) - 1
    anc = anc.to(H.DEV)
    out = torch.zeros(rows, Hq * hd, dtype=torch.bfloat16, device=H.DEV)
    fn = getattr(B.lib, "_ZN2ht18launch_attn_causalEPKvS1_S1_iiiNS_7TreeDevEiiiPvP12ihipStream_tS1_S1_iS3_")
    fn.restype = C.c_int
    fn.argtypes = [C.c_void_p] * 3 + [C.c_int] * 3 + [Tree] + [C.c_int] * 3 + [C.c_void_p] * 4 + [C.c_int, C.c_void_p]
    print("causal attention over 600 rows", flush=True)
    assert fn(q.data_ptr(), k.data_ptr(), v.data_ptr(), cap, 0, rows, Tree(None, None, None, anc.data_ptr()), Hq, Hkv, hd,
              out.data_ptr(), torch.cuda.current_stream().cuda_stream, None, None, 0, None) == 0
    torch.cuda.synchronize()
    want = torch.ones(hd, dtype=torch.float64)
    want[1] = 2.0
    err = (out.cpu().double().view(rows, Hq, hd) / want - 1).abs().amax((1, 2))
    # one bf16 rounding of the result (2^-9 relative) and of the probabilities of the first 64 keys (2^-9 of at most 1 each)
    bound = 2.0 ** -9 * (1 + 64 / torch.arange(1, rows + 1, dtype=torch.float64))
    assert bool((err <= bound).all()), (int((err - bound).argmax()), float(err.max()))

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

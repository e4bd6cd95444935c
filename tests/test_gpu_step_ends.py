"""What a step does in front of its first block and behind its last one: the tokens put together in the launch that starts the
pass, the logits stored where the caller wants them, arg-max and selection in one launch.  Needs a real MI355X.

Whole numbers are compared exactly with the rules applied to the logits that the call returned."""
import threading
import time

import numpy as np
import pytest
import torch

import gpu_harness as H
from ht_inputs import WORKLOADS, make_weights, prune_tree
from oracle import ht_oracle as O
from helpers import prompt_of, torch_dtype

pytestmark = pytest.mark.gpu

B = H.B


def _model(wl, fused, T):
    tensors = make_weights(wl, wl.seed, H.DEV, torch_dtype(wl))
    parent, rank = prune_tree(wl.branching, T)
    m = B.HTModel(B.make_config(wl, max_tree=T + len(fused) * wl.k), tensors, H.DEV)
    m.ht_set_tree(parent, rank)
    m.ht_set_fused_nodes(fused)
    m.ht_prefill(prompt_of(wl))
    return m, parent, rank


def _top(row, b):
    """The first b ids by (value descending, id ascending)."""
    return np.lexsort((np.arange(row.size), -row))[:b]


# vocabularies of one stage, of one to four, five to sixteen and more entries a lane in the first of two, of up to and more
# than the rows that are requested whole; passes below and above 128 rows; arg-max and selection in a launch each (64 nodes of up to 8
# candidates) and, with 40 draft rows of up to 4, in one
@pytest.mark.parametrize("base,vocab,T,every", [("tiny_bf16", 4112, 20, True), ("tiny_bf16", 40000, 20, True),
                                                ("tiny_bf16", 1024, 8, False), ("tiny_bf16", 2064, 8, True), ("tiny_bf16", 12304, 8, False),
                                                ("tiny_bf16", 32768, 7, True), ("tiny_bf16", 32784, 6, True),
                                                ("tiny_bf16", 131088, 5, False), ("tiny", 4096, 8, True), ("tiny_bf16", 4112, 64, True)])
def test_logits_choices_and_tokens_of_a_step(base, vocab, T, every):
    wl = WORKLOADS[base].with_(vocab=vocab, branching=(8, 7) if T > 20 else (4, 4) if T > 8 else (2, 2, 2)[:2] if T <= 7 else (3, 2), tree_size=T, max_cache=256)
    fused = list(range(T)) if every else [0, 1]
    m, parent, rank = _model(wl, fused, T)
    tokens = torch.arange(3, 3 + T, dtype=torch.int32, device=H.DEV) * 7 % vocab
    # a path of the tree that greedy decoding takes, down to a leaf, over last children
    children = [[v for v in range(1, T) if parent[v] == u] for u in range(T)]
    chosen, g = [0], torch.full((T,), -1, dtype=torch.int32, device=H.DEV)
    while children[chosen[-1]]:
        m.ht_tree_verify_step(tokens, g)
        child = children[chosen[-1]][-1]
        tokens[child] = g[chosen[-1]]
        chosen.append(child)
    m.ht_prefill(prompt_of(wl))
    seen = []
    for offset in (0, 1):                    # floats past a 16-byte address: the caller's rows stored by the head, or copied
        raw = torch.full((T * vocab + 8,), 5.0, device=H.DEV)
        z = raw[offset:offset + T * vocab].view(T, vocab)
        g = torch.full((T,), -1, dtype=torch.int32, device=H.DEV)
        print(f"step of {T} nodes, {len(fused)} drafting, vocabulary {vocab}, offset {offset}", flush=True)
        m.ht_tree_verify_step(tokens, g, z)
        torch.cuda.synchronize()
        zz = z.cpu().numpy()
        assert np.isfinite(zz).all() and bool((raw[offset + T * vocab:] == 5.0).all()) and bool((raw[:offset] == 5.0).all())
        assert np.array_equal(g.cpu().numpy(), zz.argmax(1))
        assert torch.equal(m.ht_get_buffer(B.HT_BUF_TREE_TOKENS)[:T], tokens)
        drafts = m.ht_get_buffer(B.HT_BUF_FUSED_DRAFT_LOGITS).cpu().numpy()
        cand = m.ht_get_buffer(B.HT_BUF_FUSED_CANDIDATES).cpu().numpy()
        depth = [0] * T
        for v in range(1, T):
            depth[v] = depth[parent[v]] + 1
        for f in range(len(fused)):
            for i in range(wl.k):
                width = max([rank[v] + 1 for v in range(T) if depth[v] == i + 1], default=0)
                assert np.array_equal(cand[f, i, :width], _top(drafts[f * wl.k + i], width)), (f, i)
        seen.append((zz, drafts[:len(fused) * wl.k].copy()))
        count, emitted, nxt, path = m.ht_accept_and_compact()
        toks, greedy = tokens.tolist(), zz.argmax(1).tolist()
        want, want_next = O.accept_walk(parent, toks, greedy)
        assert len(want) >= len(chosen) and want[0] == 0
        assert (path, count, nxt) == (want, len(want), want_next) and emitted == [toks[v] for v in want]
        m.ht_prefill(prompt_of(wl))          # the same step again
    assert np.array_equal(seen[0][0], seen[1][0]) and np.array_equal(seen[0][1], seen[1][1])


@pytest.mark.parametrize("base", ["tiny", "tiny_bf16"])
@pytest.mark.parametrize("fused", [[], [0]])
def test_tokens_of_the_tree_follow_its_rule(base, fused):
    """Tokens from the draft pass's candidates and from those of the pass before: the root, and cand[depth - 1][rank]."""
    wl = WORKLOADS[base]
    T = wl.tree_size
    m, parent, rank = _model(wl, fused, T)
    depth = [0] * T
    for v in range(1, T):
        depth[v] = depth[parent[v]] + 1
    in_pass = None
    for step in range(4):
        print(f"tokens of step {step} of {base}, drafting in the pass: {fused}", flush=True)
        root = int(m.ht_get_buffer(B.HT_BUF_ROOT)[0])
        if in_pass is None:
            m.ht_transfer()
        m.ht_tree_verify_step()
        torch.cuda.synchronize()
        cand = in_pass if in_pass is not None else m.ht_get_buffer(B.HT_BUF_CANDIDATES).cpu().numpy()
        want = [root] + [int(cand[depth[v] - 1][rank[v]]) for v in range(1, T)]
        assert m.ht_get_buffer(B.HT_BUF_TREE_TOKENS)[:T].cpu().tolist() == want
        drafted = m.ht_get_buffer(B.HT_BUF_FUSED_CANDIDATES).cpu().numpy().copy() if fused else None
        path = m.ht_accept_and_compact()[3]
        in_pass = drafted[fused.index(path[-1])] if fused and path[-1] in fused else None


# the sum of squares over a fraction of a workgroup, one round of 256, 512 and 1024 threads and, above 16384, a second one; pseudo rows
# that start a pass of their own
@pytest.mark.parametrize("base,d", [("tiny_bf16", 256), ("tiny_t123_bf16", 320), ("tiny_bf16", 4096), ("tiny_bf16", 8192),
                                    ("tiny_bf16", 16384), ("tiny_bf16", 16448)])
def test_first_norm_in_the_launch_that_starts_the_pass(base, d):
    """A table on 8 bytes has its rows normalised where they are read, one 2 bytes past that by the norm's own launch: same bits."""
    wl = WORKLOADS[base].with_(d_model=d)
    got = []
    for offset in (0, 1):
        tensors = make_weights(wl, wl.seed, H.DEV, torch_dtype(wl))
        raw = torch.empty(tensors["tok_emb"].numel() + 8, dtype=torch.bfloat16, device=H.DEV)
        table = raw[offset:offset + tensors["tok_emb"].numel()].view(tensors["tok_emb"].shape)
        table.copy_(tensors["tok_emb"])
        tensors["tok_emb"] = table
        parent, rank = prune_tree(wl.branching, wl.tree_size)
        m = B.HTModel(B.make_config(wl), tensors, H.DEV)
        m.ht_set_tree(parent, rank)
        m.ht_prefill(prompt_of(wl))
        print(f"first norm of {base}, d = {d}, table offset {offset}", flush=True)
        z = torch.empty(wl.tree_size, wl.vocab, device=H.DEV)
        steps = []
        for _ in range(2):
            m.ht_transfer()
            m.ht_tree_verify_step(None, None, z)
            torch.cuda.synchronize()
            steps.append(z.cpu().numpy().copy())
            steps.append(m.ht_get_buffer(B.HT_BUF_DRAFT_LOGITS).cpu().numpy().copy())
            m.ht_accept_and_compact()
        got.append(steps)
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("base", ["tiny", "tiny_bf16"])
def test_tokens_and_logits_that_are_not_this_device_s_memory(base):
    """Tokens in host memory, pageable and pinned, and 2 bytes past a word; logits into host memory: the runtime's copies take
    them, and a kernel never gets such an address."""
    wl = WORKLOADS[base]
    T = wl.tree_size
    m, _, _ = _model(wl, [0], T)
    tokens = torch.arange(3, 3 + T, dtype=torch.int32) * 7 % wl.vocab
    raw = torch.zeros(4 * T + 4, dtype=torch.uint8, device=H.DEV)
    raw[2:2 + 4 * T] = tokens.to(H.DEV).view(torch.uint8)
    on_device = tokens.to(H.DEV)
    z, zh = torch.zeros(T, wl.vocab, device=H.DEV), torch.zeros(T, wl.vocab).pin_memory()
    g = torch.zeros(T, dtype=torch.int32, device=H.DEV)
    seen = []
    for name, t, out in (("device", on_device, z), ("pageable", tokens, z), ("pinned", tokens.pin_memory(), z),
                         ("off a word", raw.data_ptr() + 2, z), ("logits to the host", on_device, zh)):
        print(f"{base}: {name}", flush=True)
        ptr = t if isinstance(t, int) else t.data_ptr()
        z.zero_()
        B._check(B.lib.ht_tree_verify_step(m.handle, ptr, g.data_ptr(), out.data_ptr(), B._stream_ptr()))
        torch.cuda.synchronize()
        assert torch.equal(m.ht_get_buffer(B.HT_BUF_TREE_TOKENS)[:T], on_device)
        seen.append((out.cpu().clone(), g.cpu().clone()))
        assert torch.isfinite(seen[-1][0]).all() and torch.equal(seen[-1][1].long(), seen[-1][0].argmax(1))
        m.ht_accept_and_compact()
        m.ht_prefill(prompt_of(wl))
    for zz, gg in seen[1:]:
        assert torch.equal(zz, seen[0][0]) and torch.equal(gg, seen[0][1])


def _busy(ms):
    """Some `ms` of products on the current stream; returns once they are enqueued."""
    a = torch.randn(4096, 4096, device=H.DEV).bfloat16()
    c = torch.empty_like(a)
    torch.mm(a, a, out=c)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(10):
        torch.mm(a, a, out=c)
    torch.cuda.synchronize()
    for _ in range(int(ms / ((time.perf_counter() - t) * 100)) + 1):
        torch.mm(a, a, out=c)


def _decode(m, steps, stream):
    out = []
    for _ in range(steps):
        m.ht_transfer(stream=stream)
        m.ht_tree_verify_step(stream=stream)
        out.append(m.ht_accept_and_compact(stream=stream))
    return out


@pytest.mark.parametrize("ms", [3, 60])
def test_acceptance_behind_other_work(ms):
    """A step with milliseconds of products in front of it on its stream: within the time that the host looks for the state, and
    beyond, where it waits for the stream."""
    wl = WORKLOADS["tiny_bf16"]
    m, _, _ = _model(wl, [], wl.tree_size)
    want = _decode(m, 2, None)
    m.ht_prefill(prompt_of(wl))
    for k in range(2):
        print(f"step {k} behind {ms} ms of products", flush=True)
        _busy(ms)
        m.ht_transfer()
        m.ht_tree_verify_step()
        start = time.perf_counter()
        assert m.ht_accept_and_compact() == want[k]
        if k:
            assert time.perf_counter() - start > ms * 5e-4


def test_two_models_on_two_threads_and_streams():
    wl = WORKLOADS["tiny_bf16"]
    models = [_model(wl, [], wl.tree_size)[0] for _ in range(2)]
    want = _decode(models[0], 12, None)
    got, streams = [None, None], [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()

    def work(i):
        for _ in range(4):
            models[i].ht_prefill(prompt_of(wl), stream=streams[i])
            got[i] = _decode(models[i], 12, streams[i])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    print("two threads", flush=True)
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got[0] == want and got[1] == want


def test_models_freed_right_behind_the_acceptance():
    wl = WORKLOADS["tiny_bf16"]
    want = None
    for k in range(6):
        print(f"model {k}", flush=True)
        m, _, _ = _model(wl, [], wl.tree_size)
        got = _decode(m, 1, None)
        m.close()
        want = want or got
        assert got == want
    torch.cuda.synchronize()

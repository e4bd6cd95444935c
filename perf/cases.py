"""What the library is timed on: calls that a program decoding with hidden transfer makes, through the public binding.

Six kinds of call:

  generate  a whole request on the fp32 model of the test configurations: prompt, then draft / verify / accept steps.
            Everything is small, so launches and latency decide.
  step      one decode step of a bf16 model at real widths over a filled cache: verify pass of a T-node tree (T = 1: plain
            autoregressive decoding) with no node, the rank-0 chain or every node drafting inside the pass, then the
            acceptance.  The tree's tokens come from an external drafter, so the numbers do not hang on near-ties of random
            logits.  A few layers stand for the whole depth: every layer costs the same, and roundings travel less far.
  prefill   the prompt of a request, into the cache.
  train     the forward pass of the training stage with its loss, all positions in one pass per block.
  attention the tree-attention call on its own (rotary, append, attention), with the tree uploaded beforehand.
  product   one projection on packed weights: the plain skinny product, or gate/up with its SiLU.
  choose    candidate log-probabilities and the tree chosen from them.

Weights, prompts and activations are random at the scales of a trained model (matrices N(0, 0.02^2), gains around 1).
"""
import heapq
import math

import torch

import paper_2404_12022_amd.binding as B

_7B = dict(d=4096, heads=32, kv_heads=32, head_dim=128, ffn=11008, vocab=32000)
_13B = dict(d=5120, heads=40, kv_heads=40, head_dim=128, ffn=13824, vocab=32000)
_70B = dict(d=8192, heads=64, kv_heads=8, head_dim=128, ffn=28672, vocab=32000)
_TINY = dict(d=256, heads=4, kv_heads=4, head_dim=64, ffn=688, vocab=1024)
_EPS, _BASE = 1e-5, 10000.0


def _room(n):
    """Decode steps that fit the cache before a step case starts its next request."""
    return max(256, n // 2)


def listed():
    return [
        # the fp32 test configuration end to end: the smallest calls there are, and the schedule that drafts after accepting
        dict(name="generate_tiny_f32", kind="generate", layers=2, k=2, n=32, tree=8, steps=16, **_TINY),
        # plain autoregressive decoding, what every verify pass is measured against
        dict(name="one_token_7b", kind="step", layers=4, k=3, n=512, tree=1, drafting="none", **_7B),
        # the ordinary step: a 64-node tree, the rank-0 chain drafts inside the pass
        dict(name="step_7b", kind="step", layers=4, k=3, n=512, tree=64, drafting="chain", **_7B),
        # the paper's own schedule, every node drafts inside the pass: 256 rows
        dict(name="step_7b_every_node", kind="step", layers=4, k=3, n=512, tree=64, drafting="all", **_7B),
        # grouped heads, a long cache and the largest matrices
        dict(name="step_70b", kind="step", layers=2, k=4, n=4096, tree=64, drafting="chain", **_70B),
        # the prompt of an ordinary request
        dict(name="prefill_7b", kind="prefill", layers=4, k=3, n=512, **_7B),
        # a long prompt of ragged length on the middle model
        dict(name="prefill_13b_long", kind="prefill", layers=3, k=3, n=1987, **_13B),
        # the training stage's forward pass at the length it is benchmarked on
        dict(name="train_7b", kind="train", layers=4, k=3, n=2048, step=1, **_7B),
        # the attention call at the size of its benchmark
        dict(name="attention_op", kind="attention", n=4096, tree=128, heads=32, kv_heads=32, head_dim=128, dtype="bf16"),
        # ... and at the size of a short chat on a small model
        dict(name="attention_small", kind="attention", n=40, tree=8, heads=4, kv_heads=4, head_dim=64, dtype="bf16"),
        # the down projection of the middle model for an odd number of rows
        dict(name="product_13b_down", kind="product", rows=33, out=5120, inner=13824, gated=False),
        # the choice of a tree from the drafts of one step
        dict(name="choose_tree", kind="choose", k=3, candidates=10, tree=64, vocab=32000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng):
    """Widths between a small model's and the middle one's; head counts and widths that fill nothing evenly among them."""
    if rng.random() < 0.3:
        return dict(rng.choice([_7B, _13B]))
    hd = rng.choice([64, 128, 128])
    kv = _log(rng, 2, 40 * 128 // hd)
    group = rng.choice([1, 1, 1, 2, 4, 8])
    while kv * group * hd > 5120:
        kv, group = max(1, kv // 2), max(1, group // 2)
    d = 16 * _log(rng, 32, 320)
    return dict(d=d, heads=kv * group, kv_heads=kv, head_dim=hd, ffn=16 * _log(rng, 64, 864), vocab=16 * _log(rng, 64, 2000))


def draw(rng):
    kind = rng.choice(["generate", "step", "step", "step", "prefill", "prefill", "train", "attention", "attention", "product",
                       "product", "choose"])
    if kind == "generate":
        return dict(kind=kind, layers=rng.randint(2, 3), k=rng.randint(1, 3), n=rng.randint(5, 60), tree=rng.randint(2, 12),
                    steps=rng.randint(4, 16), **_TINY)
    if kind == "step":
        k = rng.randint(1, 4)
        drafting = rng.choice(["none", "chain", "chain", "all"])
        tree = rng.choice([1, _log(rng, 2, 128), _log(rng, 16, 64)])
        if drafting == "all":
            tree = min(tree, 256 // (1 + k))
        if drafting == "chain":
            tree = max(tree, k + 1)
        if k == 1:
            tree = min(tree, 1 + B.HT_MAX_TOPK)          # one level holds no more candidates
        return dict(kind=kind, layers=rng.randint(2, 4), k=k, n=_log(rng, 24, 4096), tree=tree, drafting=drafting, **_shape(rng))
    if kind == "prefill":
        return dict(kind=kind, layers=rng.randint(2, 3), k=rng.randint(1, 4), n=_log(rng, 3, 2500), **_shape(rng))
    if kind == "train":
        k = rng.randint(1, 3)
        return dict(kind=kind, layers=rng.randint(2, 3), k=k, n=_log(rng, 32, 2048), step=rng.randint(1, k), **_shape(rng))
    if kind == "attention":
        if rng.random() < 0.25:          # fp32 belongs to the small model
            return dict(kind=kind, n=rng.randint(0, 300), tree=rng.randint(1, 12), heads=4, kv_heads=rng.choice([1, 2, 4]),
                        head_dim=64, dtype="f32")
        kv = rng.choice([4, 5, 8, 8, 32, 40])
        group = rng.choice([1, 1, 2, 4, 8]) if kv <= 8 else 1
        return dict(kind=kind, n=_log(rng, 16, 6000), tree=_log(rng, 1, 256), heads=kv * group, kv_heads=kv,
                    head_dim=rng.choice([64, 128, 128]), dtype="bf16")
    if kind == "product":
        gated = rng.random() < 0.5
        return dict(kind=kind, rows=_log(rng, 1, 256), out=16 * _log(rng, 40, 864), inner=8 * _log(rng, 80, 1728), gated=gated)
    k = rng.randint(1, 8)
    b = rng.randint(2, 40)
    room = sum(b ** e for e in range(k + 1))
    return dict(kind="choose", k=k, candidates=b, tree=min(_log(rng, 2, 128), room), vocab=_log(rng, 1000, 128000))


# ------------------------------------------------------------------------------------------------------------- inputs
def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _rng(seed):
    return torch.Generator(device=_device()).manual_seed(seed)


def _normal(g, shape, dtype, sigma=1.0, mean=0.0):
    return torch.empty(shape, dtype=dtype, device=_device()).normal_(mean, sigma, generator=g)


def _transfer_layer(c):
    return max(1, c["layers"] * 3 // 4)


def _weights(c, g, dtype):
    d, qd, kvd, f, v, L = c["d"], c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["ffn"], c["vocab"], c["layers"]
    w = {"tok_emb": _normal(g, (v, d), dtype, 0.02), "final_norm": _normal(g, (d,), dtype, 0.02, 1.0),
         "lm_head": _normal(g, (v, d), dtype, 0.02)}
    for name, shape in (("wq", (qd, d)), ("wk", (kvd, d)), ("wv", (kvd, d)), ("wo", (d, qd)), ("w_gate", (f, d)),
                        ("w_up", (f, d)), ("w_down", (d, f))):
        w[name] = [_normal(g, shape, dtype, 0.02) for _ in range(L)]
    for name in ("attn_norm", "ffn_norm"):
        w[name] = [_normal(g, (d,), dtype, 0.02, 1.0) for _ in range(L)]
    w["w_transfer"] = [_normal(g, (d, d), dtype, 0.02) for _ in range(c["k"])]
    return w


def _config(c, dtype, max_cache, rows):
    cfg = B.ht_config()
    cfg.n_layers, cfg.d_model, cfg.n_heads, cfg.n_kv_heads = c["layers"], c["d"], c["heads"], c["kv_heads"]
    cfg.head_dim, cfg.d_ffn, cfg.vocab, cfg.k = c["head_dim"], c["ffn"], c["vocab"], c["k"]
    cfg.rms_eps, cfg.rope_base = _EPS, _BASE
    cfg.dtype = B.HT_F32 if dtype == torch.float32 else B.HT_BF16
    for i in range(c["k"]):
        cfg.transfer_layer[i] = _transfer_layer(c)
    cfg.max_cache, cfg.max_tree = (max_cache + 7) // 8 * 8, rows
    return cfg


def _tree(size, k):
    """A complete b-ary tree of at most k levels below the root, numbered level by level: (parent, rank, depth, b)."""
    b = 1
    while sum(b ** e for e in range(k + 1)) < size:
        b += 1
    parent = [-1] + [(v - 1) // b for v in range(1, size)]
    rank = [0] + [(v - 1) % b for v in range(1, size)]
    depth = [0] * size
    for v in range(1, size):
        depth[v] = depth[parent[v]] + 1
    return parent, rank, depth, b


def _random_parents(size, seed):
    """A random tree of depth at most 6, as the attention call takes it."""
    g = torch.Generator().manual_seed(seed)
    parent, depth = [-1], [0]
    for v in range(1, size):
        p = int(torch.randint(0, v, (1,), generator=g))
        while depth[p] >= 6:
            p = parent[p]
        parent.append(p)
        depth.append(depth[p] + 1)
    return parent


def _drafting_nodes(c):
    if c["drafting"] == "none":
        return []
    if c["drafting"] == "all":
        return list(range(c["tree"]))
    parent = _tree(c["tree"], c["k"])[0]
    chain = [0]
    while len(chain) <= c["k"] and chain[-1] in parent:
        chain.append(parent.index(chain[-1]))
    return chain


def _tokens(c, g, count):
    return torch.randint(0, c["vocab"], (count,), generator=g, device=_device(), dtype=torch.int32)


def _caches(model, c):
    return [model.ht_get_buffer(which, l) for l in range(c["layers"]) for which in (B.HT_BUF_K_CACHE, B.HT_BUF_V_CACHE)]


def prepare(case, seed):
    c, g, dev = case, _rng(seed), _device()
    kind = c["kind"]
    if kind == "generate":
        prompt = _tokens(c, g, c["n"]).tolist()
        cap = c["n"] + c["steps"] * (c["k"] + 1) + c["tree"]
        model = B.HTModel(_config(c, torch.float32, cap, max(c["tree"], c["k"])), _weights(c, g, torch.float32), dev)
        parent, rank, _, _ = _tree(c["tree"], c["k"])
        model.ht_set_tree(parent, rank)
        logits = torch.zeros(c["steps"], c["tree"], c["vocab"], device=dev)
        return dict(case=c, model=model, prompt=prompt, logits=logits)
    if kind == "step":
        prompt = _tokens(c, g, c["n"]).tolist()
        tokens = _tokens(c, g, c["tree"])
        nodes = _drafting_nodes(c)
        rows = max(c["tree"] + len(nodes) * c["k"], c["k"])
        model = B.HTModel(_config(c, torch.bfloat16, c["n"] + rows + _room(c["n"]), rows), _weights(c, g, torch.bfloat16), dev)
        model.ht_set_tree(*_tree(c["tree"], c["k"])[:2])
        model.ht_set_fused_nodes(nodes)
        model.ht_prefill(prompt)
        logits = torch.zeros(c["tree"], c["vocab"], device=dev)
        drafts = model.ht_get_buffer(B.HT_BUF_FUSED_DRAFT_LOGITS) if nodes else None
        return dict(case=c, model=model, prompt=prompt, tokens=tokens, rows=rows, logits=logits, drafts=drafts, kv=_caches(model, c))
    if kind == "prefill":
        prompt = _tokens(c, g, c["n"]).tolist()
        model = B.HTModel(_config(c, torch.bfloat16, c["n"] + 128, 64), _weights(c, g, torch.bfloat16), dev)
        return dict(case=c, model=model, prompt=prompt, kv=_caches(model, c), source=model.ht_get_buffer(B.HT_BUF_TRANSFER_SRC))
    if kind == "train":
        tokens = _tokens(c, g, c["n"]).tolist()
        model = B.HTModel(_config(c, torch.bfloat16, c["n"], 64), _weights(c, g, torch.bfloat16), dev)
        need = B.C.c_size_t(0)
        B._check(B.lib.ht_training_workspace_bytes(B.C.byref(model.cfg), c["n"], B.C.byref(need)))
        ws = torch.empty(need.value, dtype=torch.uint8, device=dev)
        hidden = torch.zeros(c["n"], c["vocab"], device=dev)
        pseudo = torch.zeros(c["n"] - c["step"] + 1, c["vocab"], device=dev)
        return dict(case=c, model=model, tokens=tokens, ws=ws, hidden=hidden, pseudo=pseudo)
    if kind == "attention":
        s = _attention_inputs(c, g)
        T, Hq, hd = c["tree"], c["heads"], c["head_dim"]
        dt = s["q"].dtype
        s["out"] = torch.zeros(T, Hq * hd, dtype=dt, device=dev)
        s["scratch"] = torch.zeros(B.ht_tree_attention_scratch_bytes(T, Hq, hd), dtype=torch.uint8, device=dev)
        s["case"], s["code"] = c, B.HT_F32 if dt == torch.float32 else B.HT_BF16
        _attention_call(s, _random_parents(T, T))            # a serving loop uploads its tree once
        return s
    if kind == "product":
        M, N, K = c["rows"], c["out"], c["inner"]
        s = dict(case=c, **_product_inputs(c, g))
        if c["gated"]:
            s["packed"] = torch.zeros(B.ht_weight_pack_bytes(2 * N, K), dtype=torch.uint8, device=dev)
            B.ht_gate_up_pack(s["w"][0], s["w"][1], N, K, s["packed"])
            s["out"] = torch.zeros(M, N, dtype=torch.bfloat16, device=dev)
        else:
            s["packed"] = torch.zeros(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=dev)
            B.ht_weight_pack(s["w"], N, K, s["packed"])
            s["out"] = torch.zeros(M, N, device=dev)
            s["scratch"] = torch.empty(B.ht_skinny_gemm_scratch_bytes(M, N, K), dtype=torch.uint8, device=dev)
        return s
    d, cand, root = _choose_inputs(c, g)
    i32 = dict(dtype=torch.int32, device=dev)
    T = c["tree"]
    return dict(case=c, d=d, cand=cand, root=root, lp=torch.zeros(c["k"], B.HT_MAX_TOPK, device=dev), parent=torch.zeros(T, **i32),
                depth=torch.zeros(T, **i32), rank=torch.zeros(T, **i32), tokens=torch.zeros(T, **i32),
                anc=torch.zeros(T, B.HT_MAX_ROWS // 64, dtype=torch.int64, device=dev))


def _padded(tokens, c):
    """The emitted tokens, -1 up to the most that the steps can emit."""
    return torch.tensor(tokens + [-1] * (c["steps"] * (c["k"] + 1) - len(tokens)))


def _attention_inputs(c, g):
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    T, Hq, Hkv, hd = c["tree"], c["heads"], c["kv_heads"], c["head_dim"]
    cap = (c["n"] + T + 64 + 7) // 8 * 8
    return dict(cap=cap, q=_normal(g, (T, Hq, hd), dt), k=_normal(g, (T, Hkv, hd), dt), v=_normal(g, (T, Hkv, hd), dt),
                k_cache=_normal(g, (cap, Hkv, hd), dt), v_cache=_normal(g, (Hkv, hd, cap), dt))


def _attention_call(s, parent):
    c = s["case"]
    B.ht_tree_attention(s["q"], s["k"], s["v"], s["k_cache"], s["v_cache"], s["cap"], c["n"], c["tree"], parent, c["heads"],
                        c["kv_heads"], c["head_dim"], s["code"], _BASE, s["out"], s["scratch"])


def _product_inputs(c, g):
    M, N, K = c["rows"], c["out"], c["inner"]
    a = torch.zeros(B.ht_padded_rows(M), K, dtype=torch.bfloat16, device=_device())
    a[:M] = _normal(g, (M, K), torch.bfloat16)
    w = [_normal(g, (N, K), torch.bfloat16, 0.02) for _ in range(2 if c["gated"] else 1)]
    return dict(a=a, w=w if c["gated"] else w[0])


def _choose_inputs(c, g):
    d = _normal(g, (c["k"], c["vocab"]), torch.float32, 2.0)
    cand = torch.zeros(c["k"], B.HT_MAX_TOPK, dtype=torch.int32, device=_device())
    cand[:, :c["candidates"]] = torch.topk(d, c["candidates"], dim=1).indices.to(torch.int32)
    return d, cand, _tokens(c, g, 1)


# ---------------------------------------------------------------------------------------------------------- one pass
def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "generate":
        model, emitted = s["model"], []
        model.ht_prefill(s["prompt"])
        for i in range(c["steps"]):
            model.ht_transfer()
            model.ht_tree_verify_step(None, None, s["logits"][i])
            emitted += model.ht_accept_and_compact()[1]
        return {"logits": s["logits"], "tokens": _padded(emitted, c)}
    if kind == "step":
        model = s["model"]
        if model.ht_cache_len() + s["rows"] > model.cfg.max_cache:        # the cache is full: the next request
            model.ht_prefill(s["prompt"])
        model.ht_tree_verify_step(s["tokens"], None, s["logits"])
        accepted = model.ht_accept_and_compact()[0]
        return {"logits": s["logits"], "drafts": s["drafts"], "kv": s["kv"], "accepted": accepted}
    if kind == "prefill":
        s["model"].ht_prefill(s["prompt"])
        return {"kv": s["kv"], "source": s["source"]}
    if kind == "train":
        kl, loss = s["model"].ht_training_forward_batched(c["step"], s["tokens"], s["hidden"], s["pseudo"], s["ws"])
        return {"kl": torch.tensor(kl), "loss": loss, "hidden": s["hidden"], "pseudo": s["pseudo"]}
    if kind == "attention":
        _attention_call(s, None)
        return {"out": s["out"], "k_cache": s["k_cache"], "v_cache": s["v_cache"]}
    if kind == "product":
        if c["gated"]:
            B.ht_gate_up_silu_packed(s["a"], s["packed"], c["rows"], c["out"], c["inner"], s["out"])
        else:
            B.ht_skinny_gemm_packed(s["a"], s["packed"], c["rows"], c["out"], c["inner"], s["out"], s["scratch"])
        return s["out"]
    B.ht_candidate_logprobs(s["d"], s["cand"], c["candidates"], s["lp"])
    B.ht_dynamic_tree(s["lp"], s["cand"], s["root"], c["k"], c["candidates"], c["tree"], s["parent"], s["depth"], s["rank"],
                      s["anc"], s["tokens"])
    return {n: s[n] for n in ("lp", "parent", "depth", "rank", "anc", "tokens")}


# ------------------------------------------------------------------------------------------------ work and tolerances
def work(case):
    c, kind = case, case["kind"]
    if kind == "attention":
        T, e = c["tree"], 4 if c["dtype"] == "f32" else 2
        qd, kvd = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
        return {"bytes": e * (2 * c["n"] * kvd + 2 * T * qd + 4 * T * kvd), "flops": 4 * T * (c["n"] + 4) * qd}
    if kind == "product":
        M, N, K = c["rows"], c["out"], c["inner"]
        n = 2 * N if c["gated"] else N
        return {"bytes": 2 * n * K + 2 * M * K + M * N * (2 if c["gated"] else 4), "flops": 2 * M * n * K}
    if kind == "choose":
        return {"bytes": 4 * c["k"] * c["vocab"] + 4 * c["k"] * c["candidates"] + 48 * c["tree"], "flops": 3 * c["k"] * c["vocab"]}
    e = 4 if kind == "generate" else 2
    d, qd, kvd, v, L, t = c["d"], c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["vocab"], c["layers"], _transfer_layer(c)
    layer = d * (qd + 2 * kvd) + qd * d + 3 * d * c["ffn"]
    if kind == "step":
        T, extra, n = c["tree"], len(_drafting_nodes(c)) * c["k"], c["n"]
        maps = c["k"] * d * d if extra else 0
        rows = T * L + extra * (L - t)                            # (row, layer) pairs
        return {"bytes": e * (L * (layer + 2 * n * kvd) + v * d + maps + T * d + 2 * rows * kvd) + 4 * (T + extra) * v,
                "flops": 2 * rows * layer + 4 * rows * n * qd + 2 * (T + extra) * v * d + 2 * extra * d * d}
    if kind == "prefill":
        n = c["n"]
        return {"bytes": e * (L * (layer + 2 * n * kvd) + v * d + n * d), "flops": 2 * n * L * layer + 2 * L * n * n * qd + 2 * v * d}
    if kind == "train":
        n, P = c["n"], c["n"] - c["step"] + 1
        rows = n * L + P * (L - t)
        return {"bytes": e * (L * layer + v * d + d * d + n * d) + 4 * (n + P) * v,
                "flops": 2 * rows * layer + 2 * rows * n * qd + 2 * (n + P) * v * d + 2 * P * d * d}
    n, T, k = c["n"], c["tree"], c["k"]                           # generate: prompt, then draft and verify passes
    per = (T * L + k * (L - t)) * layer + (T + k) * v * d + k * d * d
    once = L * layer + v * d
    return {"bytes": e * (once + c["steps"] * ((L + L - t) * layer + 2 * v * d + k * d * d + 2 * L * n * kvd)) + 4 * c["steps"] * T * v,
            "flops": 2 * n * L * layer + 2 * c["steps"] * per}


def tolerance(case):
    """Against float64 the bf16 model is off by 1.5e-2 (logits after four blocks), the bf16 attention call by 3e-3, the gated
    product by 1.7e-3, the fp32 paths by 3e-7 and less; stated is up to four times that, and 3e-2 at most."""
    kind = case["kind"]
    if kind == "generate":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    if kind in ("step", "prefill", "train"):
        return {"rel": 0.03, "max": 0.3}
    if kind == "attention":
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 0.01, "max": 0.1}
    if kind == "product":
        return {"rel": 0.01, "max": 0.05} if case["gated"] else {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}


# ------------------------------------------------------------------------------------------- the same, plainly, in 64 bits
class _Plain:
    """The decoder in float64: textbook products, explicit masks, a cache that is a list of tensors."""

    def __init__(self, c, w):
        self.c, self.w = c, w
        self.k, self.v = [None] * c["layers"], [None] * c["layers"]

    def norm(self, x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + _EPS) * gain.double()

    def block(self, l, x, pos, mask, past):
        """Block l over rows x at positions pos; row i sees the first `past` cache entries and the rows of mask[i]."""
        c, w = self.c, self.w
        H, Hk, hd = c["heads"], c["kv_heads"], c["head_dim"]
        u = self.norm(x, w["attn_norm"][l])
        q = _rotate((u @ w["wq"][l].double().T).view(-1, H, hd), pos)
        k = _rotate((u @ w["wk"][l].double().T).view(-1, Hk, hd), pos)
        v = (u @ w["wv"][l].double().T).view(-1, Hk, hd)
        keys = torch.cat([self.k[l][:past], k]) if past else k
        vals = torch.cat([self.v[l][:past], v]) if past else v
        self.k[l], self.v[l] = keys, vals
        x = x + _attend(q, keys, vals, past, mask) @ w["wo"][l].double().T
        u = self.norm(x, w["ffn_norm"][l])
        g, up = u @ w["w_gate"][l].double().T, u @ w["w_up"][l].double().T
        return x + (g / (1 + torch.exp(-g)) * up) @ w["w_down"][l].double().T

    def logits(self, x):
        return self.norm(x, self.w["final_norm"]) @ self.w["lm_head"].double().T

    def prompt(self, tokens):
        """Fills the cache; returns (residual of the last token after the transfer layer, its logits)."""
        n = len(tokens)
        x = self.w["tok_emb"][torch.tensor(tokens, device=_device())].double()
        pos, mask = torch.arange(n, device=_device()), torch.ones(n, n, dtype=torch.bool, device=_device()).tril()
        for l in range(self.c["layers"]):
            if l == _transfer_layer(self.c):
                source = x[-1].clone()
            x = self.block(l, x, pos, mask, 0)
        return source, self.logits(x[-1:])[0]

    def tree(self, tokens, parent, depth, n, nodes=()):
        """A tree pass over n cached tokens with k pseudo rows under each of `nodes`: (logits, residuals after t blocks)."""
        c, T, k = self.c, len(parent), self.c["k"]
        parent, depth = list(parent), list(depth)
        for f in nodes:
            for i in range(k):
                parent.append(f if i == 0 else len(parent) - 1)
                depth.append(depth[f] + i + 1)
        mask = _ancestors(parent)
        pos = n + torch.tensor(depth, device=_device())
        x = self.w["tok_emb"][tokens.long()].double()
        for l in range(c["layers"]):
            if l == _transfer_layer(c):
                saved = x.clone()
                new = [self.w["w_transfer"][i].double() @ x[f] for f in nodes for i in range(k)]
                if new:
                    x = torch.cat([x, torch.stack(new)])
            r = x.shape[0]
            x = self.block(l, x, pos[:r], mask[:r, :r], n)
        return self.logits(x), saved

    def draft(self, source, n):
        """k pseudo rows of one source as a chain behind n cached tokens: their logits."""
        k = self.c["k"]
        x = torch.stack([self.w["w_transfer"][i].double() @ source for i in range(k)])
        pos, mask = n + torch.arange(k, device=_device()), torch.ones(k, k, dtype=torch.bool, device=_device()).tril()
        for l in range(_transfer_layer(self.c), self.c["layers"]):
            x = self.block(l, x, pos, mask, n)
        return self.logits(x)


def _rotate(x, pos):
    half = x.shape[-1] // 2
    freq = _BASE ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    angle = (pos.double()[:, None] * freq)[:, None, :]
    co, si, a, b = torch.cos(angle), torch.sin(angle), x[..., :half], x[..., half:]
    return torch.cat([a * co - b * si, b * co + a * si], dim=-1)


def _attend(q, keys, vals, past, mask):
    """softmax(q.k / sqrt(hd)) v, one head at a time; row i sees keys[:past] and keys[past + j] where mask[i, j]."""
    rows, H, hd = q.shape
    group = H // keys.shape[1]
    seen = torch.cat([torch.ones(rows, past, dtype=torch.bool, device=q.device), mask], dim=1)
    out = torch.empty(rows, H, hd, dtype=torch.float64, device=q.device)
    for h in range(H):
        s = q[:, h] @ keys[:, h // group].T.contiguous() / math.sqrt(hd)
        out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), dim=1) @ vals[:, h // group].contiguous()
    return out.reshape(rows, H * hd)


def _ancestors(parent):
    mask = torch.zeros(len(parent), len(parent), dtype=torch.bool)
    for v, p in enumerate(parent):
        if p >= 0:
            mask[v] = mask[p]
        mask[v, v] = True
    return mask.to(_device())


def _plain_caches(p, c, cap):
    """The caches as the library lays them out, zero where nothing was written."""
    out = []
    for l in range(c["layers"]):
        rows = p.k[l].shape[0]
        k = torch.zeros(cap, c["kv_heads"], c["head_dim"], dtype=torch.float64, device=_device())
        v = torch.zeros(c["kv_heads"], c["head_dim"], cap, dtype=torch.float64, device=_device())
        k[:rows] = p.k[l]
        v[:, :, :rows] = p.v[l].permute(1, 2, 0)
        out += [k, v]
    return out


def exact(case, seed):
    c, g, kind = case, _rng(seed), case["kind"]
    if kind == "generate":
        return _exact_generate(c, g)
    if kind == "step":
        prompt, tokens, nodes = _tokens(c, g, c["n"]).tolist(), _tokens(c, g, c["tree"]), _drafting_nodes(c)
        rows = max(c["tree"] + len(nodes) * c["k"], c["k"])
        p = _Plain(c, _weights(c, g, torch.bfloat16))
        p.prompt(prompt)
        parent, _, depth, _ = _tree(c["tree"], c["k"])
        z, _ = p.tree(tokens, parent, depth, c["n"], nodes)
        cap = (c["n"] + rows + _room(c["n"]) + 7) // 8 * 8
        return {"logits": z[:c["tree"]], "drafts": z[c["tree"]:] if nodes else None, "kv": _plain_caches(p, c, cap),
                "accepted": None}
    if kind == "prefill":
        prompt = _tokens(c, g, c["n"]).tolist()
        p = _Plain(c, _weights(c, g, torch.bfloat16))
        source, _ = p.prompt(prompt)
        return {"kv": _plain_caches(p, c, (c["n"] + 128 + 7) // 8 * 8), "source": source}
    if kind == "train":
        return _exact_train(c, g)
    if kind == "attention":
        s = _attention_inputs(c, g)
        n, T = c["n"], c["tree"]
        parent = _random_parents(T, T)
        depth = [0] * T
        for v in range(1, T):
            depth[v] = depth[parent[v]] + 1
        pos = n + torch.tensor(depth, device=_device())
        kc, vc = s["k_cache"].double(), s["v_cache"].double()
        kc[n:n + T] = _rotate(s["k"].double(), pos)
        vc[:, :, n:n + T] = s["v"].double().permute(1, 2, 0)
        keys, vals = kc[:n + T], vc[:, :, :n + T].permute(2, 0, 1)
        out = _attend(_rotate(s["q"].double(), pos), keys, vals, n, _ancestors(parent))
        return {"out": out, "k_cache": kc, "v_cache": vc}
    if kind == "product":
        s = _product_inputs(c, g)
        a = s["a"][:c["rows"]].double()
        if not c["gated"]:
            return a @ s["w"].double().T
        gate, up = a @ s["w"][0].double().T, a @ s["w"][1].double().T
        return gate / (1 + torch.exp(-gate)) * up
    d, cand, _ = _choose_inputs(c, g)
    lp = torch.zeros(c["k"], B.HT_MAX_TOPK, dtype=torch.float64, device=_device())
    b = c["candidates"]
    lp[:, :b] = torch.log_softmax(d.double(), dim=1).gather(1, cand[:, :b].long())
    parent, depth, rank = _best_first(lp[:, :b].tolist(), c["tree"])
    return {"lp": lp, "parent": torch.tensor(parent), "depth": torch.tensor(depth), "rank": torch.tensor(rank), "anc": None,
            "tokens": None}


def _best_first(lp, size):
    """Root and the size - 1 best nodes by (summed log-probability descending, depth, rank path)."""
    parent, depth, rank = [-1], [0], [0]
    heap = [(-lp[0][0], 1, (0,), 0, 0.0)]
    while len(parent) < size:
        score, e, path, p, base = heapq.heappop(heap)
        v = len(parent)
        parent.append(p), depth.append(e), rank.append(path[-1])
        r = path[-1] + 1
        if r < len(lp[0]):
            heapq.heappush(heap, (base - lp[e - 1][r], e, path[:-1] + (r,), p, base))
        if e < len(lp):
            heapq.heappush(heap, (score - lp[e][0], e + 1, path + (0,), v, score))
    return parent, depth, rank


def _exact_generate(c, g):
    prompt = _tokens(c, g, c["n"]).tolist()
    p = _Plain(c, _weights(c, g, torch.float32))
    source, z = p.prompt(prompt)
    root, n = int(z.argmax()), c["n"]
    parent, rank, depth, b = _tree(c["tree"], c["k"])
    logits, emitted = [], []
    for _ in range(c["steps"]):
        picks = torch.topk(p.draft(source, n), b, dim=1).indices.tolist()
        tokens = [root] + [picks[depth[v] - 1][rank[v]] for v in range(1, c["tree"])]
        z, saved = p.tree(torch.tensor(tokens, device=_device()), parent, depth, n)
        logits.append(z)
        best, cur, path = z.argmax(1).tolist(), 0, [0]
        while True:
            nxt = [v for v in range(cur + 1, c["tree"]) if parent[v] == cur and tokens[v] == best[cur]]
            if not nxt:
                break
            cur = nxt[0]
            path.append(cur)
        emitted += [tokens[v] for v in path]
        keep = list(range(n)) + [n + v for v in path]
        p.k, p.v = [k[keep] for k in p.k], [v[keep] for v in p.v]
        root, source, n = best[cur], saved[cur], n + len(path)
    return {"logits": torch.stack(logits), "tokens": _padded(emitted, c)}


def _exact_train(c, g):
    n, i, t = c["n"], c["step"], _transfer_layer(c)
    P = n - i + 1
    dev = _device()
    tokens = _tokens(c, g, n)
    p = _Plain(c, _weights(c, g, torch.bfloat16))
    x = p.w["tok_emb"][tokens.long()].double()
    pos = torch.arange(n, device=dev)
    mask = torch.ones(n, n, dtype=torch.bool, device=dev).tril()
    for l in range(c["layers"]):
        if l == t:                        # pseudo row j at position j + i sees the hidden rows 0 .. j + i - 1 and itself
            x = torch.cat([x, x[:P] @ p.w["w_transfer"][i - 1].double().T])
            both = torch.zeros(n + P, n + P, dtype=torch.bool, device=dev)
            both[:n, :n] = mask
            both[n:, :n] = torch.arange(n, device=dev)[None, :] < torch.arange(P, device=dev)[:, None] + i
            both[n:, n:] = torch.eye(P, dtype=torch.bool, device=dev)
            mask, pos = both, torch.cat([pos, torch.arange(P, device=dev) + i])
        x = p.block(l, x, pos, mask, 0)
    z = p.logits(x)
    terms = n - i - 1
    lp = torch.log_softmax(z, dim=1)
    a, b = lp[n:n + terms], lp[i:i + terms]
    kl = (a.exp() * (a - b)).sum(1)
    return {"kl": kl, "loss": float(kl.sum()), "hidden": z[:n], "pseudo": z[n:]}

"""The attention call on up to 16 rows, which rotates, appends and attends in one launch, against float64 and against the
general route (taken for rows that do not lie on 16 bytes).  Needs a real MI355X.

Caches bit for bit (both routes round the same float32 products once); outputs within the attention call's tolerance: bf16
probabilities and values, 2^-9 relative each, and float32 sums: 1e-2 in the 2-norm."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BASE = 10000.0


def _B():
    import paper_2404_12022_amd.binding as B
    return B


def say(msg):
    print(msg, flush=True)


def _parents(T, seed):
    g = torch.Generator().manual_seed(seed)
    return [-1] + [int(torch.randint(max(0, v - 3), v, (1,), generator=g)) for v in range(1, T)]


def _reference(q, k, v, kc, vc, n, parent, Hq, Hkv, hd):
    T = len(parent)
    depth, seen = [0] * T, torch.zeros(T, T, dtype=torch.bool)
    for r in range(T):
        if parent[r] >= 0:
            depth[r] = depth[parent[r]] + 1
            seen[r] = seen[parent[r]]
        seen[r, r] = True
    pos = n + torch.tensor(depth, dtype=torch.float64)
    freq = BASE ** (-torch.arange(hd // 2, dtype=torch.float64) / (hd // 2))
    angle = (pos[:, None] * freq)[:, None, :]
    co, si = torch.cos(angle), torch.sin(angle)

    def rot(x):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * co - b * si, b * co + a * si], dim=-1)

    q, k, v = (t.double().cpu() for t in (q, k, v))
    keys = torch.cat([kc[:n].double().cpu(), rot(k)])
    vals = torch.cat([vc[:, :, :n].double().cpu().permute(2, 0, 1), v])
    mask = torch.cat([torch.ones(T, n, dtype=torch.bool), seen], dim=1)
    qr, out = rot(q), torch.empty(T, Hq, hd, dtype=torch.float64)
    for h in range(Hq):
        s = (qr[:, h] @ keys[:, h // (Hq // Hkv)].T / math.sqrt(hd)).masked_fill(~mask, -math.inf)
        out[:, h] = torch.softmax(s, dim=1) @ vals[:, h // (Hq // Hkv)]
    return out.reshape(T, Hq * hd)


def _call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd, out=None):
    out = torch.zeros(T, Hq * hd, dtype=torch.bfloat16, device=DEV) if out is None else out
    scratch = torch.zeros(B.ht_tree_attention_scratch_bytes(T, Hq, hd), dtype=torch.uint8, device=DEV)
    kc, vc = kc.clone(), vc.clone()
    B.ht_tree_attention(q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd, B.HT_BF16, BASE, out, scratch)
    torch.cuda.synchronize()
    return out, kc, vc


def _off(t):
    """The same values 8 bytes past a 16-byte boundary: the general route."""
    raw = torch.zeros(t.numel() + 4, dtype=t.dtype, device=t.device)
    raw[4:] = t.flatten()
    return raw[4:].view(t.shape)


@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 15, 16])
@pytest.mark.parametrize("Hq,Hkv,hd", [(4, 4, 64), (8, 1, 64), (6, 3, 128), (32, 32, 128)])
def test_one_launch_agrees_with_the_general_route_and_with_float64(T, Hq, Hkv, hd):
    B = _B()
    for n in (0, 1, 31, 32, 33, 40, 127, 700, 1300):
        say(f"attention in one launch T={T} heads={Hq}/{Hkv}x{hd} n={n}")
        g = torch.Generator(device=DEV).manual_seed(T * 1000 + n)
        cap = (n + T + 7) // 8 * 8                                # no room behind the last row
        mk = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()
        q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
        kc[n:], vc[:, :, n:] = float("nan"), float("nan")         # slots that nobody wrote
        parent = _parents(T, n)
        out, k1, v1 = _call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
        ref_out, k2, v2 = _call(B, _off(q), k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
        assert torch.equal(k1[:n + T], k2[:n + T]) and torch.equal(v1[:, :, :n + T], v2[:, :, :n + T])
        assert torch.isnan(k1[n + T:]).all() and torch.isnan(v1[:, :, n + T:]).all()
        want = _reference(q, k, v, kc, vc, n, parent, Hq, Hkv, hd)
        err = float((out.double().cpu() - want).norm() / want.norm())
        err2 = float((ref_out.double().cpu() - want).norm() / want.norm())
        say(f"  error {err:.2e}, general route {err2:.2e}")
        assert err <= 1e-2 and err2 <= 1e-2 and err <= 1.2 * err2 + 1e-4


def test_rows_that_are_stored_to_take_the_general_route():
    """In place: `out` over q, k_new in the very cache slots it is appended to (grouped heads)."""
    B = _B()
    T, Hq, Hkv, hd, n, cap = 8, 8, 2, 64, 24, 40
    g = torch.Generator(device=DEV).manual_seed(5)
    mk = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()
    q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
    parent = _parents(T, 1)
    say("attention call in place")
    want, k1, v1 = _call(B, _off(q), k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
    direct = _call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)[0]
    over = q.clone()
    out, _, _ = _call(B, over, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd, out=over.view(T, Hq * hd))
    assert torch.equal(out, direct)
    kc2, vc2 = kc.clone(), vc.clone()
    kc2[n:n + T] = k
    out = torch.zeros(T, Hq * hd, dtype=torch.bfloat16, device=DEV)
    scratch = torch.zeros(B.ht_tree_attention_scratch_bytes(T, Hq, hd), dtype=torch.uint8, device=DEV)
    B.ht_tree_attention(q, kc2[n:n + T], v, kc2, vc2, cap, n, T, parent, Hq, Hkv, hd, B.HT_BF16, BASE, out, scratch)
    torch.cuda.synchronize()
    assert torch.equal(kc2, k1) and torch.equal(vc2, v1)
    assert torch.equal(out, want)


@pytest.mark.parametrize("which", ["k", "v", "both"])
def test_caches_off_a_16_byte_address_take_the_general_route(which):
    """Caches that are views 8 bytes past a 16-byte address: what the general route gives, bit for bit (its sums meet in
    another order than the one launch's, so some values tell the two apart)."""
    B = _B()
    T, Hq, Hkv, hd, n, cap = 9, 8, 4, 128, 77, 88
    g = torch.Generator(device=DEV).manual_seed(11)
    mk = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()
    q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
    parent = _parents(T, 1)
    say(f"attention call, offset cache: {which}")
    want, k1, v1 = _call(B, _off(q), k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
    assert not torch.equal(_call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)[0], want)
    kc2, vc2 = _off(kc) if which != "v" else kc.clone(), _off(vc) if which != "k" else vc.clone()
    out = torch.zeros(T, Hq * hd, dtype=torch.bfloat16, device=DEV)
    scratch = torch.zeros(B.ht_tree_attention_scratch_bytes(T, Hq, hd), dtype=torch.uint8, device=DEV)
    B.ht_tree_attention(q, k, v, kc2, vc2, cap, n, T, parent, Hq, Hkv, hd, B.HT_BF16, BASE, out, scratch)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and torch.equal(kc2, k1) and torch.equal(vc2, v1)


@pytest.mark.parametrize("T,Hq,Hkv", [(144, 32, 32), (250, 64, 8), (256, 64, 64), (256, 32, 32)])
def test_rows_of_many_heads_on_either_side_of_the_table_launch(T, Hq, Hkv):
    """More than 16 rows: 576 and 1024 row blocks times q and k heads of 128 (the most) work their rotary factors out for
    themselves, 1152 and 2048 read them from the table of a launch of its own.  Appended keys are float32 products rounded once: at most half a bf16 unit,
    2^-8 relative."""
    B = _B()
    n, hd, cap = 40, 128, 304
    g = torch.Generator().manual_seed(T)
    mk = lambda *s: torch.randn(*s, generator=g).to(DEV).bfloat16()
    q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
    parent = _parents(T, T)
    out, kc1, vc1 = _call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
    want = _reference(q, k, v, kc, vc, n, parent, Hq, Hkv, hd)
    err = (out.double().cpu() - want).norm() / want.norm()
    say(f"{T} rows of {Hq} + {Hkv} heads: error {err:.2e}")
    assert err <= 1e-2
    assert torch.equal(vc1[:, :, n:n + T], v.permute(1, 2, 0)) and torch.equal(kc1[:n], kc[:n])
    assert torch.equal(kc1[n + T:], kc[n + T:]) and torch.equal(vc1[:, :, n + T:], vc[:, :, n + T:])
    depth = [0] * T
    for r in range(1, T):
        depth[r] = depth[parent[r]] + 1
    angle = (n + torch.tensor(depth, dtype=torch.float64))[:, None] * BASE ** (-torch.arange(hd // 2, dtype=torch.float64) / (hd // 2))
    co, si = torch.cos(angle)[:, None], torch.sin(angle)[:, None]
    a, b = k.double().cpu()[..., :hd // 2], k.double().cpu()[..., hd // 2:]
    rot = torch.cat([a * co - b * si, b * co + a * si], dim=-1)
    assert ((kc1[n:n + T].double().cpu() - rot).abs() <= 2.0 ** -8 * rot.abs() + 1e-6).all()


@pytest.mark.parametrize("T", [9, 17, 31, 48, 63, 64, 65, 100, 127, 128])
@pytest.mark.parametrize("Hq,Hkv,hd", [(4, 4, 64), (8, 1, 64), (6, 3, 128), (32, 32, 128), (40, 5, 128)])
def test_one_launch_of_up_to_128_rows_agrees_with_the_general_route_and_with_float64(T, Hq, Hkv, hd):
    """The ring kernel on the caller's rows (up to 16 of them where many heads share long caches): own keys in tiles of 64 of
    their own, cut into slices with the cache's, which end before, at and behind a tile and an eight-key piece; shallow trees
    and a chain, as deep as a tree can be."""
    B = _B()
    for n in (0, 1, 63, 64, 72, 300, 1531):
        say(f"attention in one launch T={T} heads={Hq}/{Hkv}x{hd} n={n}")
        g = torch.Generator(device=DEV).manual_seed(T * 1000 + n)
        cap = (n + T + 7) // 8 * 8
        mk = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()
        q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
        kc[n:], vc[:, :, n:] = float("nan"), float("nan")
        parent = _parents(T, n) if n % 2 else [(r - 1) if n == 72 or r == 0 else (r - 1) // 3 for r in range(T)]
        out, k1, v1 = _call(B, q, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
        ref_out, k2, v2 = _call(B, _off(q), k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd)
        assert torch.equal(k1[:n + T], k2[:n + T]) and torch.equal(v1[:, :, :n + T], v2[:, :, :n + T])
        assert torch.isnan(k1[n + T:]).all() and torch.isnan(v1[:, :, n + T:]).all()
        want = _reference(q, k, v, kc, vc, n, parent, Hq, Hkv, hd)
        err = float((out.double().cpu() - want).norm() / want.norm())
        err2 = float((ref_out.double().cpu() - want).norm() / want.norm())
        say(f"  error {err:.2e}, general route {err2:.2e}")
        assert err <= 1e-2 and err2 <= 1e-2 and err <= 1.2 * err2 + 1e-4
        over = q.clone()
        again, _, _ = _call(B, over, k, v, kc, vc, cap, n, T, parent, Hq, Hkv, hd, out=over.view(T, Hq * hd))
        assert torch.equal(again, out)


@pytest.mark.parametrize("T,hd", [(17, 64), (64, 128), (100, 128)])
def test_depths_that_are_no_tree_s_stay_inside_the_table_of_factors(T, hd):
    """parent = NULL takes the depths as they lie in `scratch`.  Rows whose depth was written over are rotated somehow; the others
    and every value are as with the tree, and the call ends."""
    B = _B()
    Hq, Hkv, n = 4, 2, 72
    cap = (n + T + 7) // 8 * 8
    g = torch.Generator(device=DEV).manual_seed(T)
    mk = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()
    q, k, v, kc, vc = mk(T, Hq, hd), mk(T, Hkv, hd), mk(T, Hkv, hd), mk(cap, Hkv, hd), mk(Hkv, hd, cap)
    parent = [r - 1 if r < 9 else (r - 1) // 3 for r in range(T)]
    depth = [0] * T
    for r in range(1, T):
        depth[r] = depth[parent[r]] + 1
    scratch = torch.zeros(B.ht_tree_attention_scratch_bytes(T, Hq, hd), dtype=torch.uint8, device=DEV)
    out = torch.zeros(T, Hq * hd, dtype=torch.bfloat16, device=DEV)
    k1, v1, k2, v2 = kc.clone(), vc.clone(), kc.clone(), vc.clone()
    B.ht_tree_attention(q, k, v, k1, v1, cap, n, T, parent, Hq, Hkv, hd, B.HT_BF16, BASE, out, scratch)
    table = scratch.view(torch.int32)[B.HT_MAX_ROWS:2 * B.HT_MAX_ROWS]          # behind the parents
    assert table[:T].tolist() == depth
    over = {3: 1 << 30, 8: -1, T - 2: 0x7fffffff, T - 1: -(1 << 31)}
    for r, e in over.items():
        table[r] = e
    say(f"depths written over: {T} rows of {hd}")
    B.ht_tree_attention(q, k, v, k2, v2, cap, n, T, None, Hq, Hkv, hd, B.HT_BF16, BASE, out, scratch)
    torch.cuda.synchronize()
    kept = [n + r for r in range(T) if r not in over]
    assert torch.equal(k1[:n], k2[:n]) and torch.equal(k1[kept], k2[kept]) and torch.equal(v1, v2)
    assert torch.isfinite(out).all()

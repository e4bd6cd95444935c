"""The token-tiled product of passes of more than 128 rows, at the edges of its tiles, against the textbook product."""
import ctypes as C

import numpy as np
import pytest
import torch

import gpu_harness as H
from oracle import ht_oracle as O

pytestmark = pytest.mark.gpu


class Packed(C.Structure):
    _fields_ = [("p", C.c_void_p), ("N", C.c_int32), ("K", C.c_int32), ("Kp", C.c_int32)]


class RowScale(C.Structure):
    _fields_ = [("ss", C.c_void_p), ("inv_d", C.c_float), ("eps", C.c_float)]


def inputs(M, N, K, seed):
    g = torch.Generator(device=H.DEV).manual_seed(seed)
    a = torch.empty(M, K, device=H.DEV).normal_(generator=g).to(torch.bfloat16)
    w = torch.empty(N, K, device=H.DEV).normal_(0, 0.05, generator=g).to(torch.bfloat16)
    return a, w


def bound(a, w, K):
    # exact products, fp32 sums: at most K / 32 matrix steps and the splits' sums, each rounded relative to a partial sum
    # that the sum of magnitudes bounds
    return (K / 32 + 16) * 2.0 ** -24 * np.abs(H.cpu(a)) @ np.abs(H.cpu(w)).T


# rows, features and columns one below, at and one above 64, 128 and 256, odd chunk counts, one chunk, whatever tile the rule
# takes (mostly 64 x 64; the tiles one by one are below); the last: 78 tiles of 192 features in nine of 128 rows, 80 in the last
@pytest.mark.parametrize("M,N,K,splits", [(129, 16, 8, 1), (255, 240, 200, 1), (256, 256, 128, 1), (257, 272, 136, 1), (130, 144, 1032, 2),
                                          (300, 4112, 328, 1), (513, 128, 2056, 4), (1025, 528, 640, 1), (129, 2064, 4096, 8),
                                          (2047, 1040, 192, 1), (1025, 14864, 2048, 1)])
def test_token_tiled_product(M, N, K, splits):
    import paper_2404_12022_amd.binding as B
    a, w = inputs(M, N, K, M + N + K)
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    B.ht_weight_pack(w, N, K, packed)
    fn = getattr(B.lib, "_ZN2ht16launch_gemm_wideEPKvNS_7PackedWEiPfiP12ihipStream_tNS_8RowScaleE")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_int, C.c_void_p, RowScale]
    out = torch.full((splits, M, N), float("nan"), device=H.DEV)
    print(f"tiled product {M} x {N} x {K} / {splits}", flush=True)
    assert fn(a.data_ptr(), Packed(packed.data_ptr(), N, K, (K + 127) // 128 * 128), M, out.data_ptr(), splits,
              torch.cuda.current_stream().cuda_stream, RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    got = H.cpu(out.sum(0))
    assert np.all(np.abs(got - O.linear(H.cpu(a), H.cpu(w))) <= bound(a, w, K))


# every tile there is, with token rows and features left over, fewer chunks than a tile has stages and more, K splits that do
# not divide over the eight XCDs: 64 x 64, 64 x 128, 96 x 128, 128 x 128, 192 x 128, 128 x 256, 192 x 256, 256 x 256, whole
# rounds of 256 x 256 and the rest in 128 x 256
@pytest.mark.parametrize("M,N,K,splits", [(129, 1040, 136, 1), (200, 1040, 1032, 3), (200, 4112, 264, 1), (129, 3088, 1032, 2),
                                          (641, 1040, 136, 3), (200, 4112, 136, 2), (200, 5136, 136, 3), (257, 5136, 136, 2),
                                          (385, 3088, 136, 3), (641, 2064, 136, 3), (700, 6256, 392, 1), (129, 10256, 136, 3),
                                          (385, 5136, 2056, 3), (255, 32016, 136, 1), (1025, 2064, 136, 3), (511, 22032, 264, 1),
                                          (257, 10256, 136, 3), (770, 12304, 392, 1), (641, 24592, 1032, 1)])
def test_every_tile_at_its_edges(M, N, K, splits):
    import paper_2404_12022_amd.binding as B
    a, w = inputs(M, N, K, M + N + K)
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    B.ht_weight_pack(w, N, K, packed)
    fn = getattr(B.lib, "_ZN2ht16launch_gemm_wideEPKvNS_7PackedWEiPfiP12ihipStream_tNS_8RowScaleE")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_int, C.c_void_p, RowScale]
    out = torch.full((splits, M + 1, N), float("nan"), device=H.DEV).view(-1)[:splits * M * N + N]
    out[splits * M * N:] = 7.0
    stream = torch.cuda.current_stream().cuda_stream
    print(f"tiled product {M} x {N} x {K} / {splits}", flush=True)
    assert fn(a.data_ptr(), Packed(packed.data_ptr(), N, K, (K + 127) // 128 * 128), M, out.data_ptr(), splits, stream,
              RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    want = a.double() @ w.double().T
    err = (K / 32 + 16) * 2.0 ** -24 * (a.double().abs() @ w.double().abs().T)
    assert bool(((out[:splits * M * N].view(splits, M, N).sum(0).double() - want).abs() <= err).all())
    assert bool((out[splits * M * N:] == 7.0).all())
    f = N // 2 // 16 * 16
    gate, up = w[:f].contiguous(), w[f:2 * f].contiguous()
    gu = torch.empty(B.ht_weight_pack_bytes(2 * f, K), dtype=torch.uint8, device=H.DEV)
    B.ht_gate_up_pack(gate, up, f, K, gu)
    silu = getattr(B.lib, "_ZN2ht21launch_gemm_wide_siluEPKvNS_7PackedWEiPvP12ihipStream_tNS_8RowScaleE")
    silu.restype, silu.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_void_p, RowScale]
    act = torch.full((M + 1, f), 7.0, dtype=torch.bfloat16, device=H.DEV)
    assert silu(a.data_ptr(), Packed(gu.data_ptr(), 2 * f, K, (K + 127) // 128 * 128), M, act.data_ptr(), stream,
                RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    g, u = want[:, :f], want[:, f:2 * f]
    act_want = g / (1 + torch.exp(-g)) * u
    assert bool(((act[:M].double() - act_want).abs() <= 2.0 ** -8 * act_want.abs() + 1e-4 * act_want.abs().max()).all())
    assert bool((act[M] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [(33, 4112, 1032), (47, 2064, 4096), (48, 208, 200), (129, 64, 64), (160, 4096, 1024), (193, 528, 2048), (256, 1040, 4104)])
def test_packed_products_of_between_32_and_48_and_of_more_than_128_rows(M, N, K):
    """The public calls: plain product (with its K splits) and gate/up with SiLU."""
    import paper_2404_12022_amd.binding as B
    a, w = inputs(B.ht_padded_rows(M), N, K, 7 * M + N)
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    B.ht_weight_pack(w, N, K, packed)
    scratch = torch.empty(B.ht_skinny_gemm_scratch_bytes(M, N, K), dtype=torch.uint8, device=H.DEV)
    out = torch.full((M, N), float("nan"), device=H.DEV)
    B.ht_skinny_gemm_packed(a, packed, M, N, K, out, scratch)
    torch.cuda.synchronize()
    want = O.linear(H.cpu(a[:M]), H.cpu(w))
    assert np.all(np.abs(H.cpu(out) - want) <= bound(a[:M], w, K))
    f = N // 2 // 16 * 16
    gate, up = w[:f].contiguous(), w[f:2 * f].contiguous()
    gu = torch.empty(B.ht_weight_pack_bytes(2 * f, K), dtype=torch.uint8, device=H.DEV)
    B.ht_gate_up_pack(gate, up, f, K, gu)
    act = torch.full((M, f), float("nan"), dtype=torch.bfloat16, device=H.DEV)
    B.ht_gate_up_silu_packed(a, gu, M, f, K, act)
    torch.cuda.synchronize()
    want = O.silu(O.linear(H.cpu(a[:M]), H.cpu(gate))) * O.linear(H.cpu(a[:M]), H.cpu(up))
    # one bf16 rounding (half an ulp, 2^-9 relative) on values whose fp32 sums carry far smaller errors
    assert np.all(np.abs(H.cpu(act) - want) <= 2.0 ** -8 * np.abs(want) + 1e-4 * np.abs(want).max())


@pytest.mark.parametrize("M,N,K", [(129, 1040, 1032), (200, 272, 4096), (256, 4096, 264)])
@pytest.mark.parametrize("off_a,off_w", [(4, 0), (0, 4), (4, 4)])
def test_operands_that_are_not_16_byte_aligned(M, N, K, off_a, off_w):
    """Rows and packed weights 8 bytes past a 16-byte address, as a view into a larger buffer gives them."""
    import paper_2404_12022_amd.binding as B
    a0, w = inputs(B.ht_padded_rows(M), N, K, M + K)
    store = torch.zeros(a0.numel() + 8, dtype=torch.bfloat16, device=H.DEV)
    a = store[off_a:off_a + a0.numel()].view_as(a0).copy_(a0)
    want = O.linear(H.cpu(a0[:M]), H.cpu(w))

    def packed_for(rows):
        return torch.empty(B.ht_weight_pack_bytes(rows, K) + 16, dtype=torch.uint8, device=H.DEV)[2 * off_w:]

    print(f"misaligned product {M} x {N} x {K}, offsets {off_a} {off_w}", flush=True)
    packed = packed_for(N)
    B.ht_weight_pack(w, N, K, packed)
    scratch = torch.empty(B.ht_skinny_gemm_scratch_bytes(M, N, K), dtype=torch.uint8, device=H.DEV)
    for call in (lambda o: B.ht_skinny_gemm_packed(a, packed, M, N, K, o, scratch), lambda o: B.ht_skinny_gemm_packed(a, packed, M, N, K, o),
                 lambda o: B.ht_skinny_gemm_packed_noalloc(a, packed, M, N, K, o)):
        out = torch.full((M, N), float("nan"), device=H.DEV)
        call(out)
        torch.cuda.synchronize()
        assert np.all(np.abs(H.cpu(out) - want) <= bound(a0[:M], w, K))
    f = N // 2 // 16 * 16
    gate, up = w[:f].contiguous(), w[f:2 * f].contiguous()
    gu = packed_for(2 * f)
    B.ht_gate_up_pack(gate, up, f, K, gu)
    act = torch.full((M, f), float("nan"), dtype=torch.bfloat16, device=H.DEV)
    B.ht_gate_up_silu_packed(a, gu, M, f, K, act)
    torch.cuda.synchronize()
    want = O.silu(O.linear(H.cpu(a0[:M]), H.cpu(gate))) * O.linear(H.cpu(a0[:M]), H.cpu(up))
    assert np.all(np.abs(H.cpu(act) - want) <= 2.0 ** -8 * np.abs(want) + 1e-4 * np.abs(want).max())


class Segs(C.Structure):
    _fields_ = [("w", C.c_void_p * 3), ("rows", C.c_int32 * 3), ("nseg", C.c_int32)]


class Qkv(C.Structure):
    _fields_ = [(f, C.c_void_p) for f in ("cs", "q", "kc", "vc")] + [(f, C.c_int32) for f in ("n", "Hq", "Hkv", "hd", "cap")] + [
        ("n_dev", C.c_void_p), ("tail_row", C.c_int32), ("tail_n", C.c_int32), ("tail_cap", C.c_int32)] + [
        (f, C.c_void_p) for f in ("tail_cs", "tail_kc", "tail_vc")]


def factors(rows, first, hd):
    angle = (first + torch.arange(rows, dtype=torch.float64, device=H.DEV))[:, None] * 10000.0 ** (
        -torch.arange(hd // 2, dtype=torch.float64, device=H.DEV) / (hd // 2))
    return torch.stack([angle.cos(), angle.sin()], dim=2).float().contiguous()


def rotated(x, cs):
    co, si = cs[:, None, :, 0].double(), cs[:, None, :, 1].double()
    a, b = x.chunk(2, dim=2)
    return torch.cat([a * co - b * si, b * co + a * si], dim=2)


# 1800 rows, 48 tiles of 256 features: 32 in whole rounds, the last 16 as tiles of half the size; the seam, feature 8192, lies
# between two k heads (48 / 24 heads of 128) or two v heads (32 / 32)
@pytest.mark.parametrize("Hq,Hkv", [(48, 24), (32, 32)])
@pytest.mark.parametrize("tail", [0, 1100])
def test_rotary_and_append_across_the_two_launches_of_a_product(Hq, Hkv, tail):
    import paper_2404_12022_amd.binding as B
    M, K, hd, n = 1800, 2048, 128, 5
    qd, kvd = Hq * hd, Hkv * hd
    N = qd + 2 * kvd
    assert N == 12288
    a, w = inputs(M, N, K, Hq + tail)
    lib, s = B.lib, torch.cuda.current_stream().cuda_stream
    repack = getattr(lib, "_ZN2ht13launch_repackENS_10WeightSegsEiiiPvP12ihipStream_t")
    repack.restype, repack.argtypes = C.c_int, [Segs] + [C.c_int] * 3 + [C.c_void_p] * 2
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    parts = [w[:qd], w[qd:qd + kvd], w[qd + kvd:]]
    assert repack(Segs((C.c_void_p * 3)(*[p.data_ptr() for p in parts]), (C.c_int32 * 3)(qd, kvd, kvd), 3), K, 2, hd, packed.data_ptr(), s) == 0
    own = tail or M                                   # rows with the first caches; the others have caches of their own
    cap, tail_n = n + M + 3, 2
    cap, tail_cap = (cap + 7) // 8 * 8, 808
    cs, tail_cs = factors(M, n, hd), factors(M, 3, hd)
    bf = dict(dtype=torch.bfloat16, device=H.DEV)
    q = torch.full((M, Hq, hd), 7.0, **bf)
    kc, vc = torch.full((cap, Hkv, hd), 7.0, **bf), torch.full((Hkv, hd, cap), 7.0, **bf)
    tk, tv = torch.full((tail_cap, Hkv, hd), 7.0, **bf), torch.full((Hkv, hd, tail_cap), 7.0, **bf)
    qe = Qkv(cs.data_ptr(), q.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, Hq, Hkv, hd, cap, None, tail, tail_n, tail_cap,
             tail_cs.data_ptr() if tail else None, tk.data_ptr() if tail else None, tv.data_ptr() if tail else None)
    fn = getattr(lib, "_ZN2ht20launch_gemm_wide_qkvEPKvNS_7PackedWEiNS_11QkvEpilogueEP12ihipStream_tNS_8RowScaleE")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, Qkv, C.c_void_p, RowScale]
    print(f"q|k|v over two launches, {Hq}/{Hkv} heads, tail {tail}", flush=True)
    assert fn(a.data_ptr(), Packed(packed.data_ptr(), N, K, K), M, qe, s, RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    y = a.double() @ w.double().T
    err = (K / 32 + 16) * 2.0 ** -24 * float((a.double().abs() @ w.double().abs().T).max())

    def close(got, want):                             # one bf16 rounding (half an ulp, 2^-9) on sums that are off by err
        return bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 4 * err).all())

    both = torch.cat([cs[:own], tail_cs[:M - own]])
    assert close(q, rotated(y[:, :qd].view(M, Hq, hd), both))
    k = rotated(y[:, qd:qd + kvd].reshape(M, Hkv, hd), both)
    v = y[:, qd + kvd:].reshape(M, Hkv, hd)
    assert close(kc[n:n + own], k[:own]) and close(vc[:, :, n:n + own].permute(2, 0, 1), v[:own])
    assert bool((kc[:n] == 7).all()) and bool((kc[n + own:] == 7).all()) and bool((vc[:, :, :n] == 7).all()) and bool((vc[:, :, n + own:] == 7).all())
    if tail:
        t1 = tail_n + M - own
        assert close(tk[tail_n:t1], k[own:]) and close(tv[:, :, tail_n:t1].permute(2, 0, 1), v[own:])
        assert bool((tk[:tail_n] == 7).all()) and bool((tk[t1:] == 7).all()) and bool((tv[:, :, t1:] == 7).all())


# 512 rows: 192 x 128 tiles, 300 and 129 rows: smaller ones.  At 512 rows six of 2.6 million keys once came out of the other order.
@pytest.mark.parametrize("M,Hq,Hkv,hd,K", [(512, 32, 32, 128, 4096), (300, 32, 8, 64, 1024), (129, 8, 8, 96, 512)])
def test_rotary_products_are_rounded_in_one_order(M, Hq, Hkv, hd, K):
    """Every rotated value, bit for bit: low half fma(a, cos, -(b sin)), high half fma(b, cos, a sin) of the plain product's
    sums, whatever tile multiplied the row."""
    import paper_2404_12022_amd.binding as B
    n, qd, kvd = 3, Hq * hd, Hkv * hd
    N, cap = qd + 2 * kvd, (n + M + 7) // 8 * 8
    a, w = inputs(M, N, K, M + hd)
    lib, s = B.lib, torch.cuda.current_stream().cuda_stream
    repack = getattr(lib, "_ZN2ht13launch_repackENS_10WeightSegsEiiiPvP12ihipStream_t")
    repack.restype, repack.argtypes = C.c_int, [Segs] + [C.c_int] * 3 + [C.c_void_p] * 2
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    parts = [w[:qd], w[qd:qd + kvd], w[qd + kvd:]]
    assert repack(Segs((C.c_void_p * 3)(*[p.data_ptr() for p in parts]), (C.c_int32 * 3)(qd, kvd, kvd), 3), K, 2, hd, packed.data_ptr(), s) == 0
    weights = Packed(packed.data_ptr(), N, K, (K + 127) // 128 * 128)
    bf = dict(dtype=torch.bfloat16, device=H.DEV)
    q, kc, vc = torch.zeros(M, Hq, hd, **bf), torch.zeros(cap, Hkv, hd, **bf), torch.zeros(Hkv, hd, cap, **bf)
    cs = factors(M, n, hd)
    fn = getattr(lib, "_ZN2ht20launch_gemm_wide_qkvEPKvNS_7PackedWEiNS_11QkvEpilogueEP12ihipStream_tNS_8RowScaleE")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, Qkv, C.c_void_p, RowScale]
    print(f"order of the rotary products {M} x {N} x {K}", flush=True)
    qe = Qkv(cs.data_ptr(), q.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, Hq, Hkv, hd, cap, None, 0, 0, 0, None, None, None)
    assert fn(a.data_ptr(), weights, M, qe, s, RowScale(None, 0.0, 0.0)) == 0
    plain = getattr(lib, "_ZN2ht16launch_gemm_wideEPKvNS_7PackedWEiPfiP12ihipStream_tNS_8RowScaleE")
    plain.restype, plain.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_int, C.c_void_p, RowScale]
    sums = torch.empty(M, N, device=H.DEV)
    assert plain(a.data_ptr(), weights, M, sums.data_ptr(), 1, s, RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    # packed order of a head: eight features, then their eight partners
    x = sums[:, :qd + kvd].view(M, Hq + Hkv, hd // 16, 2, 8)
    low, high = x[:, :, :, 0].reshape(M, Hq + Hkv, hd // 2), x[:, :, :, 1].reshape(M, Hq + Hkv, hd // 2)
    co, si = cs[:, None, :, 0], cs[:, None, :, 1]
    fma = lambda p, f, c: (p.double() * f.double() + c.double()).float()
    want = torch.cat([fma(low, co, -(high * si)), fma(high, co, low * si)], dim=2).to(torch.bfloat16)
    assert torch.equal(q, want[:, :Hq]) and torch.equal(kc[n:n + M], want[:, Hq:])


def test_gate_up_across_the_two_launches_of_a_product():
    import paper_2404_12022_amd.binding as B
    M, f, K = 1800, 6144, 2048                        # 48 tiles of 256 interleaved features, the seam at 4096 of 6144
    a, w = inputs(M, 2 * f, K, 11)
    packed = torch.empty(B.ht_weight_pack_bytes(2 * f, K), dtype=torch.uint8, device=H.DEV)
    B.ht_gate_up_pack(w[:f].contiguous(), w[f:].contiguous(), f, K, packed)
    fn = getattr(B.lib, "_ZN2ht21launch_gemm_wide_siluEPKvNS_7PackedWEiPvP12ihipStream_tNS_8RowScaleE")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_void_p, RowScale]
    act = torch.full((M + 1, f), 7.0, dtype=torch.bfloat16, device=H.DEV)
    print("gate/up over two launches", flush=True)
    assert fn(a.data_ptr(), Packed(packed.data_ptr(), 2 * f, K, K), M, act.data_ptr(), torch.cuda.current_stream().cuda_stream,
              RowScale(None, 0.0, 0.0)) == 0
    torch.cuda.synchronize()
    gate, up = a.double() @ w[:f].double().T, a.double() @ w[f:].double().T
    want = gate / (1 + torch.exp(-gate)) * up
    assert bool(((act[:M].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-4 * want.abs().max()).all())
    assert bool((act[M] == 7).all())


# ---- each tile by its index: features and tokens
TILES = [(256, 256), (128, 256), (192, 256), (192, 128), (128, 128), (96, 128), (64, 128), (64, 64)]


def tile_launch(B):
    fn = getattr(B.lib, "_ZN2ht16launch_gemm_tileEiiPKvNS_7PackedWEiPviNS_11QkvEpilogueEP12ihipStream_t")
    fn.restype, fn.argtypes = C.c_int, [C.c_int, C.c_int, C.c_void_p, Packed, C.c_int, C.c_void_p, C.c_int, Qkv, C.c_void_p]
    return fn


@pytest.mark.parametrize("tile", range(8))
@pytest.mark.parametrize("K,splits", [(72, 1), (264, 1), (1032, 3)])
def test_tile_sums_and_gated_features_at_its_edges(tile, K, splits):
    """One tile after the other, whatever the rule would take: a row and seven more than two tiles of rows, one feature block
    more than three tiles and one less than two; two chunks, fewer than a ring holds, five, and an odd number in three splits."""
    import paper_2404_12022_amd.binding as B
    lib, stream = tile_launch(B), torch.cuda.current_stream().cuda_stream
    F, R = TILES[tile]
    for M, N in ((2 * R + 1, 3 * F + 16), (2 * R + 7, 2 * F - 16), (R - 1, F)):
        a, w = inputs(M, N, K, M + N + K)
        packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
        B.ht_weight_pack(w, N, K, packed)
        out = torch.full((splits * M * N + N,), 7.0, device=H.DEV)
        out[:splits * M * N] = float("nan")
        print(f"tile {F} x {R}: {M} x {N} x {K} / {splits}", flush=True)
        assert lib(tile, 0, a.data_ptr(), Packed(packed.data_ptr(), N, K, (K + 127) // 128 * 128), M, out.data_ptr(), splits, Qkv(), stream) == 0
        torch.cuda.synchronize()
        want = a.double() @ w.double().T
        err = (K / 32 + 16) * 2.0 ** -24 * (a.double().abs() @ w.double().abs().T)
        assert bool(((out[:splits * M * N].view(splits, M, N).sum(0).double() - want).abs() <= err).all())
        assert bool((out[splits * M * N:] == 7.0).all())
        if splits > 1:
            continue
        f = N // 32 * 16                                  # an odd number of pairs of blocks among them
        gu = torch.empty(B.ht_weight_pack_bytes(2 * f, K), dtype=torch.uint8, device=H.DEV)
        B.ht_gate_up_pack(w[:f].contiguous(), w[f:2 * f].contiguous(), f, K, gu)
        act = torch.full((M + 1, f), 7.0, dtype=torch.bfloat16, device=H.DEV)
        assert lib(tile, 1, a.data_ptr(), Packed(gu.data_ptr(), 2 * f, K, (K + 127) // 128 * 128), M, act.data_ptr(), 1, Qkv(), stream) == 0
        torch.cuda.synchronize()
        g, u = want[:, :f], want[:, f:2 * f]
        act_want = g / (1 + torch.exp(-g)) * u
        assert bool(((act[:M].double() - act_want).abs() <= 2.0 ** -8 * act_want.abs() + 1e-4 * act_want.abs().max()).all())
        assert bool((act[M] == 7.0).all())


@pytest.mark.parametrize("tile", range(8))
@pytest.mark.parametrize("hd", [32, 64, 96, 128])
def test_tile_rotates_and_appends_at_its_edges(tile, hd):
    """Five q heads, three k and three v heads: the seams between q, k and v fall inside tiles of most sizes, the borders of
    tiles of 96 and 192 features inside heads.  With and without rows that have caches of their own."""
    import paper_2404_12022_amd.binding as B
    K, n, Hq, Hkv = 136, 5, 5, 3
    M = TILES[tile][1] + 9
    qd, kvd = Hq * hd, Hkv * hd
    N = qd + 2 * kvd
    a, w = inputs(M, N, K, M + hd)
    lib, s = tile_launch(B), torch.cuda.current_stream().cuda_stream
    repack = getattr(B.lib, "_ZN2ht13launch_repackENS_10WeightSegsEiiiPvP12ihipStream_t")
    repack.restype, repack.argtypes = C.c_int, [Segs] + [C.c_int] * 3 + [C.c_void_p] * 2
    packed = torch.empty(B.ht_weight_pack_bytes(N, K), dtype=torch.uint8, device=H.DEV)
    parts = [w[:qd], w[qd:qd + kvd], w[qd + kvd:]]
    assert repack(Segs((C.c_void_p * 3)(*[p.data_ptr() for p in parts]), (C.c_int32 * 3)(qd, kvd, kvd), 3), K, 2, hd, packed.data_ptr(), s) == 0
    y = a.double() @ w.double().T
    err = (K / 32 + 16) * 2.0 ** -24 * float((a.double().abs() @ w.double().abs().T).max())
    cs, tail_cs = factors(M, n, hd), factors(M, 3, hd)
    bf = dict(dtype=torch.bfloat16, device=H.DEV)

    def close(got, want):                             # one bf16 rounding (half an ulp, 2^-9) on sums that are off by err
        return bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 4 * err).all())

    for tail in (0, M // 2 + 3):
        own = tail or M
        cap, tail_n, tail_cap = (n + M + 10) // 8 * 8, 2, (M + 10) // 8 * 8
        q = torch.full((M + 1, Hq, hd), 7.0, **bf)
        kc, vc = torch.full((cap, Hkv, hd), 7.0, **bf), torch.full((Hkv, hd, cap), 7.0, **bf)
        tk, tv = torch.full((tail_cap, Hkv, hd), 7.0, **bf), torch.full((Hkv, hd, tail_cap), 7.0, **bf)
        qe = Qkv(cs.data_ptr(), q.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, Hq, Hkv, hd, cap, None, tail, tail_n, tail_cap,
                 tail_cs.data_ptr() if tail else None, tk.data_ptr() if tail else None, tv.data_ptr() if tail else None)
        print(f"tile {TILES[tile]}: q|k|v of heads of {hd}, tail {tail}", flush=True)
        assert lib(tile, 3 if tail else 2, a.data_ptr(), Packed(packed.data_ptr(), N, K, (K + 127) // 128 * 128), M, None, 1, qe, s) == 0
        torch.cuda.synchronize()
        both = torch.cat([cs[:own], tail_cs[:M - own]])
        k, v = rotated(y[:, qd:qd + kvd].reshape(M, Hkv, hd), both), y[:, qd + kvd:].reshape(M, Hkv, hd)
        assert close(q[:M], rotated(y[:, :qd].reshape(M, Hq, hd), both)) and bool((q[M] == 7).all())
        assert close(kc[n:n + own], k[:own]) and close(vc[:, :, n:n + own].permute(2, 0, 1), v[:own])
        assert bool((kc[:n] == 7).all()) and bool((kc[n + own:] == 7).all())
        assert bool((vc[:, :, :n] == 7).all()) and bool((vc[:, :, n + own:] == 7).all())
        t1 = tail_n + M - own
        if tail:
            assert close(tk[tail_n:t1], k[own:]) and close(tv[:, :, tail_n:t1].permute(2, 0, 1), v[own:])
        first, last = (tail_n, t1) if tail else (0, 0)
        assert bool((tk[:first] == 7).all()) and bool((tk[last:] == 7).all())
        assert bool((tv[:, :, :first] == 7).all()) and bool((tv[:, :, last:] == 7).all())

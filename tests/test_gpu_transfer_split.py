"""The hidden transfer of several sources on the matrix cores, launched directly, against the fp64 product."""
import ctypes as C
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu

SYMBOL = "_ZN2ht15launch_transferEiPKfPKiiPKPKvPfiiiiPvP12ihipStream_t"


@pytest.fixture(scope="module", autouse=True)
def no_garbage_left():
    """What earlier tests left in reference cycles is freed here, not in the middle of a later test that watches the
    allocator's count."""
    yield
    gc.collect()


def launch(h, rows, F, maps, out, i0, steps, row_stride, d):
    import paper_2404_12022_amd.binding as B
    fn = getattr(B.lib, SYMBOL)
    fn.restype = C.c_int
    fn.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p] + [C.c_int] * 4 + [C.c_void_p] * 2
    scratch = torch.empty((F + 63) // 64 * 4 * 3 * ((d + 63) // 64 * 2) * 1024, dtype=torch.uint8, device="cuda:0")
    ptrs = torch.tensor([m.data_ptr() for m in maps], dtype=torch.int64, device="cuda:0")
    assert fn(B.HT_BF16, h.data_ptr(), rows.data_ptr() if rows is not None else None, F, ptrs.data_ptr(), out.data_ptr(), i0, steps,
              row_stride, d, scratch.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


# source counts around the operand forms (5 side by side; tiles of 16; 64 per workgroup), widths below one 64-column step,
# with a ragged last step, with a ragged last row block, and full size
@pytest.mark.parametrize("F,d,steps", [(2, 8, 1), (5, 24, 3), (6, 40, 2), (4, 200, 3), (16, 328, 1), (17, 136, 2), (32, 264, 1),
                                       (33, 520, 3), (64, 1032, 2), (65, 72, 1), (127, 256, 1), (5, 4096, 3), (64, 4096, 2)])
def test_transfer_of_several_sources_matches_the_fp64_product(F, d, steps):
    g = torch.Generator(device="cuda:0").manual_seed(F * 10007 + d)
    dev = "cuda:0"
    i0, images = 1, F + 3
    maps = [torch.empty(d, d, device=dev).normal_(0, 0.02, generator=g).to(torch.bfloat16) for _ in range(i0 + steps)]
    h = torch.empty(images, d, device=dev).normal_(0, 1, generator=g)
    h[:, ::7] *= 1e-4                                                   # values of unlike sizes side by side
    rows = torch.randperm(images, generator=torch.Generator().manual_seed(d))[:F].to(torch.int32).to(dev)
    row_stride = steps + 1                                              # a gap that must stay untouched
    out = torch.full((F * row_stride, d), 7.0, device=dev)
    print(f"transfer F={F} d={d} steps={steps}", flush=True)
    launch(h, rows, F, maps, out, i0, steps, row_stride, d)
    got = out.view(F, row_stride, d)
    assert bool((got[:, steps] == 7.0).all())
    src = h[rows.long()].double()
    for i in range(steps):
        w = maps[i0 + i].double()
        ref = src @ w.T
        # fp32 sums of at most d / 128 + 16 additions each, every one rounded relative to a partial sum that the sum of
        # magnitudes bounds (the products themselves are exact)
        bound = (d / 128 + 16) * 2.0 ** -24 * (src.abs() @ w.abs().T)
        assert bool(((got[:, i].double() - ref).abs() <= bound).all())


# up to five sources: one row block per workgroup up to 512 row blocks (rings of three, six and four steps), then four, three
# and two
@pytest.mark.parametrize("F,d,steps", [(2, 264, 4), (4, 1016, 4), (5, 1032, 3), (4, 1032, 4), (2, 1024, 8), (4, 2056, 8), (3, 1640, 8), (2, 4800, 8)])
def test_row_blocks_per_workgroup(F, d, steps):
    test_transfer_of_several_sources_matches_the_fp64_product(F, d, steps)


def test_infinite_and_nan_sources_stay_in_their_row():
    d, F, dev = 256, 20, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(5)
    w = torch.empty(d, d, device=dev).normal_(0, 0.02, generator=g).to(torch.bfloat16)
    w = torch.where(w == 0, torch.full_like(w, 0.01), w)                # infinity times zero would be NaN in any order
    h = torch.empty(F, d, device=dev).normal_(0, 1, generator=g)
    h[3, 17], h[5, 40], h[7, 0] = float("inf"), float("nan"), 3.0e38
    out = torch.zeros(F, d, device=dev)
    launch(h, None, F, [w], out, 0, 1, 1, d)
    ref = h.double() @ w.double().T
    assert bool((out[3] == torch.sign(w[:, 17].float()) * float("inf")).all()) and bool(out[5].isnan().all())
    ok = [i for i in range(F) if i not in (3, 5)]
    bound = (d / 128 + 16) * 2.0 ** -24 * (h[ok].double().abs() @ w.double().abs().T)
    assert bool(((out[ok].double() - ref[ok]).abs() <= bound).all())


@pytest.mark.parametrize("F", [3, 7, 20])
def test_infinite_and_nan_weights_reach_the_sums_they_belong_to(F):
    """Sources of few mantissa bits have lower pieces of zero: an infinite weight must give infinity all the same."""
    d, dev = 264, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(F)
    w = torch.empty(d, d, device=dev).normal_(0, 0.02, generator=g).to(torch.bfloat16)
    w[5, 9], w[17, 200], w[100, 3] = float("inf"), float("-inf"), float("nan")
    h = torch.empty(F, d, device=dev).normal_(0, 1, generator=g)
    h[::2] = h[::2].to(torch.bfloat16).float()
    h = torch.where(h == 0, torch.full_like(h, 0.5), h)
    out = torch.zeros(F, d, device=dev)
    launch(h, None, F, [w], out, 0, 1, 1, d)
    inf = float("inf")
    assert bool((out[:, 5] == torch.sign(h[:, 9]) * inf).all()) and bool((out[:, 17] == -torch.sign(h[:, 200]) * inf).all())
    assert bool(out[:, 100].isnan().all())
    rest = [o for o in range(d) if o not in (5, 17, 100)]
    ref = h.double() @ w[rest].double().T
    bound = (d / 128 + 16) * 2.0 ** -24 * (h.double().abs() @ w[rest].double().abs().T)
    assert bool(((out[:, rest].double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("d", [256, 1032])
def test_one_source_alone_and_among_others(d):
    """fp32 maps: the same bits however many sources share the launch.  bf16 maps, where several sources are summed in another
    order: within the fp32 rounding of the two sums."""
    import paper_2404_12022_amd.binding as B
    fn = getattr(B.lib, SYMBOL)
    fn.restype = C.c_int
    fn.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p] + [C.c_int] * 4 + [C.c_void_p] * 2
    g, dev = torch.Generator(device="cuda:0").manual_seed(d), "cuda:0"
    h = torch.empty(20, d, device=dev).normal_(0, 1, generator=g)
    scratch = torch.empty(4 * 3 * ((d + 63) // 64 * 2) * 1024, dtype=torch.uint8, device=dev)
    for dtype, code in ((torch.float32, B.HT_F32), (torch.bfloat16, B.HT_BF16)):
        w = torch.empty(d, d, device=dev).normal_(0, 0.02, generator=g).to(dtype)
        ptrs = torch.tensor([w.data_ptr()], dtype=torch.int64, device=dev)

        def run(rows):
            out = torch.zeros(rows, d, device=dev)
            assert fn(code, h.data_ptr(), None, rows, ptrs.data_ptr(), out.data_ptr(), 0, 1, 1, d, scratch.data_ptr(),
                      torch.cuda.current_stream().cuda_stream) == 0
            torch.cuda.synchronize()
            return out

        alone = run(1)
        bound = 2 * (d / 128 + 16) * 2.0 ** -24 * (h[:1].double().abs() @ w.double().abs().T)
        for rows in (3, 7, 20):
            among = run(rows)[:1]
            if dtype == torch.float32:
                assert torch.equal(alone, among)
            else:
                assert bool(((alone.double() - among.double()).abs() <= bound).all())

"""Rotary factors against sums of 64 bits of mantissa."""
import ctypes as C

import numpy as np
import pytest
import torch

import gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base", [100.0, 10000.0, 500000.0])
@pytest.mark.parametrize("hd", [64, 96, 128])
def test_factors_are_the_rounded_values(base, hd):
    """A factor is the float nearest to the exact value, unless that value lies so close to the middle between two floats that
    fp64 cannot tell: the frequency's last place (2^-52 of it) times the position, and the last place of the factor."""
    import paper_2404_12022_amd.binding as B
    rows, first, half = 5000, 7, hd // 2
    fn = getattr(B.lib, "_ZN2ht17launch_rope_tableEPfPKiiiifP12ihipStream_tS2_")
    fn.restype, fn.argtypes = C.c_int, [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_float] + [C.c_void_p] * 2
    table = torch.full((rows, half, 2), float("nan"), device=H.DEV)
    print(f"rotary factors, base {base}, heads of {hd}", flush=True)
    assert fn(table.data_ptr(), None, first, rows, hd, base, torch.cuda.current_stream().cuda_stream, None) == 0
    torch.cuda.synchronize()
    pos = first + np.arange(rows, dtype=np.longdouble)[:, None]
    angle = pos * np.longdouble(base) ** (-np.arange(half, dtype=np.longdouble) / half)
    got, want = table.cpu().numpy(), np.stack([np.cos(angle), np.sin(angle)], axis=2)
    rounded = want.astype(np.float32)
    wrong = got != rounded
    middle = (got.astype(np.longdouble) + rounded.astype(np.longdouble)) / 2
    allowed = np.broadcast_to(((pos + 1) * np.longdouble(2) ** -52)[:, :, None], want.shape)
    assert np.all(np.abs(want - middle)[wrong] <= allowed[wrong]), (int(wrong.sum()), float(np.abs(want - middle)[wrong].max()))

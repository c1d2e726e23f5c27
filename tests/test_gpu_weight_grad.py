"""The bf16 weight gradient's tiles against float64: every tile shape, token counts around the 64-row
slices and the ring of buffers (a partial slice alone, after one, after many),
widths that leave partial tiles, and split reductions, the last split partial.  Each case
names its tile (rows, columns, four slices in flight) and splits and asserts them.

Bound: a sum of M products of bf16 values in fp32, in any order, is off by at most
(M + 6) 2^-24 sum |dy| |x|."""
import pytest

from tests.gpu_util import say
from tests.test_launch_choices_cpu import weight_grad

pytestmark = pytest.mark.gpu


T64x64, T64x128 = (64, 64, False), (64, 128, False)   # (64 x 64 always has four slices in flight)
T128x128, T128x128_DEEP, T128x192 = (128, 128, False), (128, 128, True), (128, 192, False)


@pytest.mark.parametrize("M,N,K,tile,splits", [
    (1, 8, 8, T64x64, 1), (63, 72, 200, T64x64, 1), (64, 64, 64, T64x64, 1), (65, 136, 72, T64x64, 1),
    (130, 200, 1160, T64x64, 1), (257, 328, 72, T64x64, 1), (323, 8, 1152, T64x64, 1), (2000, 1152, 1152, T64x64, 1),
    (1, 4120, 456, T64x128, 1), (65, 600, 3280, T64x128, 1), (202, 4688, 392, T64x128, 1), (4250, 392, 4208, T64x128, 2),
    (1, 3808, 1552, T128x128, 1), (129, 1480, 4168, T128x128, 1), (5955, 1952, 1192, T128x128, None),
    (1065, 712, 2728, T128x128_DEEP, 1), (4097, 1152, 1152, T128x128_DEEP, 2), (4441, 4112, 208, T128x128_DEEP, None),
    (64, 3584, 1720, T128x192, 1), (4300, 4608, 576, T128x192, 2), (5001, 1152, 4616, T128x192, 1),
    (9999, 640, 3456, T128x192, 5),
])
def test_weight_gradient(M, N, K, tile, splits):
    import torch

    import paper_2403_10266_amd as dsp
    got = weight_grad(M, N, K)
    assert got[0] == tile and (got[1] == splits if splits else got[1] > 1)
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    dy, x = (torch.randn((M, c), generator=gen, device="cuda:0").to(torch.bfloat16) for c in (N, K))
    say(f"weight gradient M={M} N={N} K={K}")
    dw, _ = dsp.dsp_linear_bwd_weight(dy, x)
    a, b = dy.double().t().contiguous(), x.double()
    err = (dw.double() - a @ b).abs()
    assert bool((err <= (M + 6) * 2.0 ** -24 * (a.abs() @ b.abs())).all())
    again, _ = dsp.dsp_linear_bwd_weight(dy, x)
    assert torch.equal(dw, again)

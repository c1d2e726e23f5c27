"""The bf16 weight gradient's tiles against float64: token counts around the 64-row
slices and the ring of buffers (a partial slice alone, after one, after many),
widths that leave partial tiles, and split reductions, the last split partial.

Bound: a sum of M products of bf16 values in fp32, in any order, is off by at most
(M + 6) 2^-24 sum |dy| |x|."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 8), (63, 72, 200), (64, 64, 64), (65, 136, 72), (130, 200, 1160), (257, 328, 72), (323, 8, 1152),
    (2000, 1152, 1152), (4097, 1152, 1152), (4300, 4608, 576), (5001, 1152, 4616), (9999, 640, 3456),
])
def test_weight_gradient(M, N, K):
    import torch

    import paper_2403_10266_amd as dsp
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    dy, x = (torch.randn((M, c), generator=gen, device="cuda:0").to(torch.bfloat16) for c in (N, K))
    say(f"weight gradient M={M} N={N} K={K}")
    dw, _ = dsp.dsp_linear_bwd_weight(dy, x)
    a, b = dy.double().t().contiguous(), x.double()
    err = (dw.double() - a @ b).abs()
    assert bool((err <= (M + 6) * 2.0 ** -24 * (a.abs() @ b.abs())).all())
    again, _ = dsp.dsp_linear_bwd_weight(dy, x)
    assert torch.equal(dw, again)

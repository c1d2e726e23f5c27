"""The bf16 GEMM's tiles against float64: every tile shape (64 x 64 and 128 x 128 with four
K slices in flight, 64 x 128, 128 x 128 and 128 x 192 with two, the register-staged 256-row
tiles), as many, fewer and more K slices than buffers, partial tiles on both sides, and
each epilogue.  Each case names its tile (rows, columns, four slices in flight) and
asserts that the launch takes it; one tile for the plain GELU where two are named.

Bound per output: fp32 accumulation of K bf16 products is off by at most
(K + 4) 2^-24 sum |a| |w| (bias and residual included in the sum), the GELU
evaluation by 1e-6 of that magnitude, and a bf16 result by its rounding: half an ulp
of 8 significant bits, 2^-8 of the value."""
import pytest

import synth
from tests.gpu_util import say
from tests.test_gpu_block_bwd import _train_case
from tests.test_launch_choices_cpu import linear

pytestmark = pytest.mark.gpu


T64x64, T64x128 = (64, 64, False), (64, 128, False)   # (64 x 64 always has four slices in flight)
T128x128, T128x128_DEEP, T128x192 = (128, 128, False), (128, 128, True), (128, 192, False)


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.mark.parametrize("epi", ["none", "gelu", "relu", "resid", "f32"])
@pytest.mark.parametrize("M,N,K,tile,gelu_tile", [
    (1, 8, 64, T64x128, None), (63, 72, 128, T64x128, None), (65, 200, 192, T64x128, None),     # 1 to 5 slices, 2 buffers
    (100, 64, 256, T64x128, None), (130, 1160, 320, T64x128, None), (770, 4664, 448, T64x128, None),
    (8451, 136, 64, T64x64, None), (8668, 152, 128, T64x64, None), (8918, 144, 192, T64x64, None),  # 1 to 5, 4 buffers
    (8246, 144, 256, T64x64, None), (8373, 160, 320, T64x64, None), (65, 200, 448, T64x64, None),
    (513, 1160, 1152, T64x64, None),
    (2500, 1152, 192, T128x128, T64x128), (8268, 656, 192, T128x128, None), (4501, 3464, 1152, T128x128, None),
    (2001, 1160, 4608, T128x128_DEEP, None), (385, 4712, 4608, T128x128_DEEP, None),
    (9092, 1288, 64, T128x192, None), (6569, 1160, 320, T128x192, None), (1201, 4600, 1152, T128x192, None),
    (8001, 1160, 1152, T128x192, None),
    (8159, 1448, 4608, (256, 192, False), None), (3974, 3856, 1152, (256, 256, False), None),
    (100, 104, 72, (256, 128, False), None),
])
def test_gemm_tiles(torch, M, N, K, tile, gelu_tile, epi):
    import paper_2403_10266_amd as dsp
    assert linear(M, N, K, epi == "gelu") == (gelu_tile if gelu_tile and epi == "gelu" else tile)
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)

    def draw(*s):
        return torch.randn(s, generator=gen, device="cuda:0")

    a, w, b = (draw(*s).to(torch.bfloat16) for s in ((M, K), (N, K), (N,)))
    r = draw(M, N) if epi == "resid" else None
    code = {"none": dsp.DSP_EPI_NONE, "gelu": dsp.DSP_EPI_GELU, "relu": dsp.DSP_EPI_RELU, "resid": dsp.DSP_EPI_RESID,
            "f32": dsp.DSP_EPI_F32}[epi]
    say(f"gemm tiles M={M} N={N} K={K} {epi}")
    got = dsp.dsp_linear(a, w, b, r, code).double()
    want = a.double() @ w.double().t() + b.double()
    mag = a.double().abs() @ w.double().abs().t() + b.double().abs()
    if epi == "resid":
        want, mag = want + r.double(), mag + r.double().abs()
    bound = (K + 4) * 2.0 ** -24 * mag
    if epi == "gelu":
        want, bound = torch.nn.functional.gelu(want), 1.2 * bound + 1e-6 * (1 + want.abs())   # |GELU'| < 1.13
    elif epi == "relu":
        want = torch.relu(want)
    if epi not in ("resid", "f32"):
        bound = bound + 2.0 ** -8 * (want.abs() + bound)
    err = (got - want).abs()
    assert bool((err <= bound).all()), float((err - bound).max())


@pytest.mark.parametrize("flags,T,S", [(0, 3, 10), (4, 5, 40)])
def test_block_train_small_tiles(torch, flags, T, S):
    """Few tokens at widths that are multiples of 64: the training epilogues (kept
    pre-activation, its use in the backward) on 64-row tiles."""
    w = synth.Workload("block_64", "block", "bf16", B=2, T=T, S=S, C=128, H=2, F=256, seed=31)
    _train_case(torch, w, True, flags)


def test_block_train_kept_derivative_small_tiles(torch):
    """Tokens that fill every CU with 256-row tiles at a width of 64: GELU' is kept, and
    both it and its use in the backward run on 64-row tiles."""
    w = synth.Workload("block_kept", "block", "bf16", B=1, T=37, S=260, C=64, H=2, F=1160, seed=32)
    tokens = w.B * w.T * w.S
    assert -(-tokens // 256) * -(-w.F // 192) >= 256 and linear(tokens, w.F, w.C) == T64x128
    _train_case(torch, w, True, 0)


@pytest.mark.parametrize("offset", [1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(65, 200, 448), (130, 1160, 320), (2001, 1160, 4608), (4501, 3464, 1152),
                                   (8001, 4616, 1152), (14000, 1160, 4608), (100, 100, 72)])
def test_bias_alignment(torch, M, N, K, offset):
    """A bias that starts `offset` elements into a buffer: the bits of an aligned one."""
    import paper_2403_10266_amd as dsp
    gen = torch.Generator(device="cuda:0").manual_seed(M + offset)
    a, w, buf = (torch.randn(s, generator=gen, device="cuda:0").to(torch.bfloat16) for s in ((M, K), (N, K), (N + 4,)))
    b = buf[offset:offset + N]
    r = torch.randn((M, N), generator=gen, device="cuda:0")
    say(f"gemm bias offset={offset} M={M} N={N} K={K}")
    assert b.data_ptr() % 8 == 2 * offset
    for code, resid in ((dsp.DSP_EPI_NONE, None), (dsp.DSP_EPI_GELU, None), (dsp.DSP_EPI_RESID, r)):
        assert torch.equal(dsp.dsp_linear(a, w, b, resid, code), dsp.dsp_linear(a, w, b.clone(), resid, code)), code

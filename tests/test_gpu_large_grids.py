"""Calls whose work-groups are more than one grid takes (2^32 threads along x): very
long and narrow fp32 operands.  Every output is compared, in pieces."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

PIECE = 1 << 28


@pytest.fixture(scope="module")
def torch():
    import torch
    yield torch
    torch.cuda.empty_cache()


def _ramp(torch, n):
    """n floats that differ from place to place, exact in fp32"""
    t = torch.arange(n, device="cuda:0", dtype=torch.int32)
    return t.bitwise_and_(0xFFFF).to(torch.float32)


def _product(torch, got, column, factor):
    got, column = got.reshape(-1), column.reshape(-1)
    assert got.numel() == column.numel()
    for i in range(0, got.numel(), PIECE):
        assert torch.equal(got[i:i + PIECE], column[i:i + PIECE] * factor), i


def test_linear_f32_rows(torch):
    import paper_2403_10266_amd as dsp
    M = (1 << 30) + 65
    a = _ramp(torch, M).view(M, 1)
    say(f"linear fp32 M={M} N=1 K=1")
    _product(torch, dsp.dsp_linear(a, torch.full((1, 1), 3.0, device="cuda:0")), a, 3.0)


def test_linear_bwd_f32(torch):
    import paper_2403_10266_amd as dsp
    n = (1 << 30) + 65
    x = _ramp(torch, n)
    say(f"linear gradients fp32, {n} rows of the input gradient and columns of the weight gradient")
    _product(torch, dsp.dsp_linear_bwd_data(x.view(n, 1), torch.full((1, 1), 5.0, device="cuda:0")), x, 5.0)
    dw, _ = dsp.dsp_linear_bwd_weight(torch.full((1, 1), 7.0, device="cuda:0"), x.view(1, n))
    _product(torch, dw, x, 7.0)


def test_attention_f32_units(torch):
    """2^24 and some units of 33 rows, head width 1: forward and gradients of the units
    on both sides of the first grid's end, and of the last ones, against a run of theirs."""
    import paper_2403_10266_amd as dsp
    X, L = (1 << 24) + 40, 33
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    q, k, v, do = (torch.randn((1, X, L, 1), generator=gen, device="cuda:0") for _ in range(4))
    say(f"attention fp32 X={X} L={L} D=1")
    o, lse = dsp.dsp_attn_general(q, k, v, 1, 1, with_lse=True)
    grads = dsp.dsp_attn_general_bwd(q, k, v, o, do, lse, 1, 1)
    for x in (0, X // 2 - 100, X - 200):
        at = slice(x, x + 200)
        qs, ks, vs, ds = (t[0, at].clone()[None] for t in (q, k, v, do))
        want, wl = dsp.dsp_attn_general(qs, ks, vs, 1, 1, with_lse=True)
        wg = dsp.dsp_attn_general_bwd(qs, ks, vs, want, ds, wl, 1, 1)
        for got, w in ((o, want), (lse, wl), *zip(grads, wg)):
            assert torch.equal(got[:, at], w), x


def test_bias_gradient_f32_columns(torch):
    import paper_2403_10266_amd as dsp
    n = (1 << 27) + 17
    dy = _ramp(torch, n)
    say(f"bias gradient fp32 of {n} columns")
    _, db = dsp.dsp_linear_bwd_weight(dy.view(1, n), torch.full((1, 1), 2.0, device="cuda:0"), with_bias=True)
    _product(torch, db, dy, 1.0)

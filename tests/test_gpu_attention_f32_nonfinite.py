"""fp32 attention with infinite scores and operands: what a softmax over the row gives,
whatever the order of the keys.  The reference is torch in float64 on the CPU."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

INF = float("inf")


def _case(L, Lk, D, seed):
    import torch
    g = torch.Generator().manual_seed(seed)
    q, do = (torch.randn((1, 1, L, D), generator=g).abs() + 0.1 for _ in range(2))
    k, v = (torch.randn((1, 1, Lk, D), generator=g) for _ in range(2))
    return q, k, v, do


def _softmax(q, k, v):
    import torch
    s = q[0, 0].double() @ k[0, 0].double().t() / q.shape[-1] ** 0.5
    return torch.softmax(s, -1) @ v[0, 0].double(), torch.logsumexp(s, -1)


def _same(got, want, what):
    import torch
    got, want = got.double().cpu(), want.double()
    assert torch.equal(torch.isnan(got), torch.isnan(want)), what
    fin = torch.isfinite(want)
    assert torch.equal(got[~fin & ~torch.isnan(want)], want[~fin & ~torch.isnan(want)]), what
    assert bool(((got - want)[fin].abs() <= 1e-5 * (1 + want[fin].abs())).all()), what


@pytest.mark.parametrize("L,Lk,D,masked", [
    (40, 100, 40, range(32)), (40, 100, 128, range(32)), (7, 70, 48, range(64)), (130, 96, 16, range(1, 70)),
    (33, 64, 72, [*range(1, 32), *range(33, 64)]), (5, 20, 24, range(20)), (20, 64, 128, range(64)),
])
def test_masked_keys(L, Lk, D, masked):
    """Keys of -inf under positive queries: scores of -inf, for whole leading tiles or all keys."""
    import torch

    import paper_2403_10266_amd as dsp
    q, k, v, _ = _case(L, Lk, D, L + Lk + D)
    k[0, 0, list(masked)] = -INF
    say(f"masked keys L={L} Lk={Lk} D={D} masked={len(list(masked))}")
    o, lse = dsp.dsp_attn_general(q.cuda(), k.cuda(), v.cuda(), 1, 1, with_lse=True)
    want, wl = _softmax(q, k, v)
    _same(o[0, 0], want, "o")
    if len(list(masked)) < Lk:
        _same(lse[0, 0, 0], wl, "lse")
    else:
        assert bool(torch.isnan(lse).all())

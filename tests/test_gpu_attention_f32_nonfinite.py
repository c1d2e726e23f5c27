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


def _grads(q, k, v, o, do, lse):
    """The gradients of the general definition, row by row: P = exp(S - lse)."""
    q, k, v, o, do = (t[0, 0].double() for t in (q, k, v, o, do))
    scale = q.shape[-1] ** -0.5
    p = (q @ k.t() * scale - lse[0, 0, 0].double()[:, None]).exp()
    dz = p * (do @ v.t() - (do * o).sum(-1, keepdim=True))
    return dz @ k * scale, dz.t() @ q * scale, p.t() @ do


@pytest.mark.parametrize("L,Lk,D", [(30, 33, 40), (5, 20, 72), (35, 130, 128), (130, 35, 16)])
@pytest.mark.parametrize("what", ["key", "dout"])
def test_gradients_with_an_infinite_row(L, Lk, D, what):
    """A key of -inf (probability 0 under positive queries), or an infinite gradient row:
    the rows and keys that fill a tile up add nothing to the others' gradients."""
    import torch

    import paper_2403_10266_amd as dsp
    q, k, v, do = _case(L, Lk, D, L + Lk + D)
    v = v.abs() + 0.1
    if what == "key":
        k[0, 0, 3] = -INF
    o, lse = dsp.dsp_attn_general(q.cuda(), k.cuda(), v.cuda(), 1, 1, with_lse=True)
    if what == "dout":
        k = k.abs() + 0.1          # dQ = dZ K: one sign for the infinite row
        o, lse = dsp.dsp_attn_general(q.cuda(), k.cuda(), v.cuda(), 1, 1, with_lse=True)
        do[0, 0, 2] = INF
        o[0, 0, 2] = -1.0          # Delta of that row is -inf, so dZ is +inf there
    say(f"infinite {what} L={L} Lk={Lk} D={D}")
    got = dsp.dsp_attn_general_bwd(q.cuda(), k.cuda(), v.cuda(), o, do.cuda(), lse, 1, 1)
    want = _grads(q, k, v, o.cpu(), do, lse.cpu())
    for g, w, name in zip(got, want, ("dq", "dk", "dv")):
        _same(g[0, 0], w, name)

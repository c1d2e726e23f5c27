"""fp32 attention of many short units: the wave-per-unit and thread-per-row kernels of a
few keys, the two-wave matrix kernel of 33 to 64 rows, the narrowest padded width;
forward, row statistics and gradients against float64.

Bound: scores and sums of fp32 products, as the repository's fp32 bar (1e-5) on outputs
of order 1."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("X,H,Hkv,L,Lk,D", [
    (1, 2, 2, 3, 3, 72), (1, 2, 1, 64, 3, 64), (1, 2, 2, 65, 3, 72), (1, 2, 2, 3, 4, 72),      # few keys, few units
    (512, 4, 4, 6, 6, 72), (512, 4, 2, 7, 6, 80), (512, 4, 4, 7, 7, 80), (600, 4, 4, 64, 4, 96), (512, 4, 4, 8, 8, 32),
    (511, 4, 4, 8, 8, 16), (4100, 4, 4, 10, 10, 16), (2100, 4, 4, 33, 33, 16), (2100, 4, 4, 65, 40, 16),
    (2048, 4, 4, 4, 4, 8), (4100, 4, 4, 5, 6, 8), (2048, 4, 4, 2, 3, 40), (1024, 4, 4, 1, 2, 40), (4096, 4, 4, 2, 2, 24),
    (3, 2, 2, 33, 70, 72), (3, 2, 1, 64, 31, 100), (3, 2, 2, 64, 64, 16), (2, 2, 2, 20, 40, 15), (2, 2, 2, 130, 35, 16),
])
def test_short_units(X, H, Hkv, L, Lk, D):
    import torch

    import paper_2403_10266_amd as dsp
    gen = torch.Generator(device="cuda:0").manual_seed(L + Lk + D)
    q, do = (torch.randn((1, X, L, H * D), generator=gen, device="cuda:0") for _ in range(2))
    k, v = (torch.randn((1, X, Lk, Hkv * D), generator=gen, device="cuda:0") for _ in range(2))
    say(f"fp32 short units X={X} H={H} Hkv={Hkv} L={L} Lk={Lk} D={D}")
    o, lse = dsp.dsp_attn_general(q, k, v, H, Hkv, with_lse=True)
    grads = dsp.dsp_attn_general_bwd(q, k, v, o, do, lse, H, Hkv)

    def heads(t, n):
        t = t[0].double().view(X, -1, n, D).transpose(1, 2)
        return t.repeat_interleave(H // n, 1)
    q64, k64, v64, d64 = heads(q, H), heads(k, Hkv), heads(v, Hkv), heads(do, H)
    s = q64 @ k64.transpose(2, 3).contiguous() * D ** -0.5
    p = s.softmax(-1)
    o64 = p @ v64
    dz = p * (d64 @ v64.transpose(2, 3).contiguous() - (d64 * o64).sum(-1, keepdim=True))
    want = [dz @ k64 * D ** -0.5, dz.transpose(2, 3).contiguous() @ q64 * D ** -0.5, p.transpose(2, 3).contiguous() @ d64]

    def rows(t, n):   # sum over a group's query heads, back to (X, L, n D)
        return t.view(X, n, H // n, -1, D).sum(2).transpose(1, 2).reshape(X, -1, n * D)
    pairs = [(o[0], rows(o64, H), "o"), (lse[0], s.logsumexp(-1), "lse")]
    pairs += [(g[0], rows(w, n), name) for g, w, n, name in zip(grads, want, (H, Hkv, Hkv), ("dq", "dk", "dv"))]
    for got, w, name in pairs:
        scale = max(1.0, float(w.abs().max()))
        assert float((got.double() - w).abs().max()) <= 1e-5 * scale, name

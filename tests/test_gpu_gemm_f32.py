"""The fp32 GEMMs (dsp_linear and its gradients) at the edges of their tiles (64; K
slices of 32, split among 1, 2 or 4 groups), with sizes and pointers that allow
no 16-byte access, against float64.

Bound: a sum of K fp32 products in any order is off by at most
(K + 2) 2^-24 sum |a| |w|; 4 more roundings cover bias and residual."""
import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (63, 65, 31), (64, 64, 32), (65, 66, 33), (129, 127, 36), (5, 1152, 72), (4100, 2052, 44),
         (4097, 2049, 7), (70, 300, 1030), (600, 1300, 260), (100, 90, 2049),
         (2, 1160, 257), (3, 100, 37), (16, 200, 320), (17, 130, 70), (300, 2, 1152), (40, 16, 129), (33, 17, 900)]


def _off(a, off):
    """a on the GPU, `off` floats past a 16-byte boundary."""
    import torch
    t = torch.empty(a.size + off, dtype=torch.float32, device="cuda:0")
    v = t[off:].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


def _within(got, want, mag, K):
    err = np.abs(got.cpu().numpy().astype(np.float64) - want)
    assert (err <= (K + 6) * 2.0 ** -24 * mag + 1e-30).all(), float((err / (mag + 1e-30)).max())


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_gemm_f32(M, N, K, off):
    import paper_2403_10266_amd as dsp
    rng = np.random.default_rng(M + N + K)
    x, w, b, r, dy = (rng.standard_normal(s, dtype=np.float32) for s in ((M, K), (N, K), (N,), (M, N), (M, N)))
    say(f"fp32 gemm M={M} N={N} K={K} off={off}")
    xd, wd, bd, rd, dyd = (_off(a, off) for a in (x, w, b, r, dy))
    x6, w6, b6, r6, d6 = (a.astype(np.float64) for a in (x, w, b, r, dy))
    ax, aw, ad = np.abs(x6), np.abs(w6), np.abs(d6)
    out = _off(np.zeros((M, N), np.float32), off)
    dsp.dsp_linear(xd, wd, bd, rd, dsp.DSP_EPI_RESID, out=out)
    _within(out, x6 @ w6.T + b6 + r6, ax @ aw.T + np.abs(b6) + np.abs(r6), K)
    dx = _off(np.zeros((M, K), np.float32), off)
    dsp.dsp_linear_bwd_data(dyd, wd, out=dx)
    _within(dx, d6 @ w6, ad @ aw, N)
    dw, _ = dsp.dsp_linear_bwd_weight(dyd, xd)
    _within(dw, d6.T @ x6, ad.T @ ax, M)

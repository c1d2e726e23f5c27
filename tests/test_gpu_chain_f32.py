"""The one-kernel fp32 chain at the edges of its 16 x 16 tiles and 4-lane attention
tasks: group lengths and widths that are not multiples of 16 (zero-padded
reductions), more tasks than threads, every head width; against the fp64 oracle at
the fp32 bar."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_close, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,S,C,H", [(1, 1, 1, 8, 1), (1, 17, 3, 24, 3), (1, 5, 33, 40, 5), (1, 64, 16, 64, 8),
                                       (2, 3, 63, 56, 7), (1, 2, 64, 64, 1), (1, 31, 2, 32, 1), (1, 9, 48, 48, 3)])
@pytest.mark.parametrize("bias", [False, True])
def test_chain_tiles(B, T, S, C, H, bias):
    import paper_2403_10266_amd as dsp
    rng = np.random.default_rng(B + T + S + C + H)
    x = rng.standard_normal((B, T, S, C), dtype=np.float32)
    names = {"wqkv_s": 3 * C, "wo_s": C, "wqkv_t": 3 * C, "wo_t": C}
    p = {n: rng.standard_normal((o, C), dtype=np.float32) / np.float32(np.sqrt(C)) for n, o in names.items()}
    if bias:
        p.update({"b" + n[1:]: rng.standard_normal(o, dtype=np.float32) for n, o in names.items()})
    say(f"chain B={B} T={T} S={S} C={C} H={H} bias={bias}")
    y = dsp.dsp_st_block_forward(dev(x, "f32"), {n: dev(v, "f32") for n, v in p.items()}, H,
                                 flags=dsp.DSP_BLOCK_ATTN_ONLY)
    C3 = lambda h, w, b: h @ p[w].astype(np.float64).T + (p[b].astype(np.float64) if bias else 0.0)

    def half(v, side, attn):
        qkv = C3(v, "wqkv_" + side, "bqkv_" + side)
        return C3(attn(qkv[..., :C], qkv[..., C:2 * C], qkv[..., 2 * C:], H), "wo_" + side, "bo_" + side)

    want = half(x.astype(np.float64), "s", oracle.spatial_attention)
    want = half(oracle.switch(want, 1, 2, 1)[0], "t", oracle.temporal_attention)
    scale = max(1.0, float(np.abs(want).max()))
    assert_close(host(y) / scale, want / scale, "f32", "chain")

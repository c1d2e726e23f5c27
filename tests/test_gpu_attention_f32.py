"""fp32 attention and its gradients at the edges of the matrix-core kernels: 32-row
tiles, 32- and 128-row work-groups, head widths between the padded instances
(32, 64, 72, 96, 128) and past them, rows that allow no 16-byte access, grouped
heads; against the fp64 oracle at the fp32 bar (gradients divided by their
largest magnitude)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_close, host, say
from tests.test_gpu_attention_general import _grad_close
from tests.test_gpu_gemm_f32 import _off

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,X,Lq,Lk,H,Hkv,D,off", [
    (1, 3, 32, 32, 2, 2, 72, 0), (1, 2, 33, 31, 2, 2, 72, 0), (2, 2, 129, 65, 4, 2, 72, 1), (1, 1, 128, 256, 2, 1, 64, 0),
    (1, 2, 40, 300, 2, 2, 80, 0), (1, 2, 31, 64, 2, 2, 96, 1), (1, 1, 70, 33, 2, 2, 100, 0), (1, 1, 20, 130, 2, 1, 128, 0),
    (1, 1, 34, 40, 2, 2, 130, 0), (1, 2, 1, 1, 2, 2, 5, 0), (1, 2, 200, 40, 3, 3, 33, 0), (1, 9, 8, 8, 4, 4, 72, 0),
])
def test_attention_f32_edges(B, X, Lq, Lk, H, Hkv, D, off):
    import paper_2403_10266_amd as dsp
    rng = np.random.default_rng(Lq + 3 * Lk + D)
    q, do = (rng.standard_normal((B, X, Lq, H * D), dtype=np.float32) for _ in range(2))
    k, v = (rng.standard_normal((B, X, Lk, Hkv * D), dtype=np.float32) for _ in range(2))
    say(f"fp32 attention B={B} X={X} Lq={Lq} Lk={Lk} H={H} Hkv={Hkv} D={D} off={off}")
    qd, kd, vd, dod = (_off(a, off) for a in (q, k, v, do))
    o, lse = dsp.dsp_attn_general(qd, kd, vd, H, Hkv, out=_off(np.zeros_like(q), off), with_lse=True)
    assert_close(host(o), oracle.attention_grouped(q, k, v, H, Hkv), "f32", "o")
    grads = dsp.dsp_attn_general_bwd(qd, kd, vd, o, dod, lse, H, Hkv, *(_off(np.zeros_like(a), off) for a in (q, k, v)))
    for got, w, name in zip(grads, oracle.attention_grouped_bwd(q, k, v, do, H, Hkv), ("dq", "dk", "dv")):
        if np.abs(w).max() < 1e-12:      # one key: dq = dk = 0 up to fp32 rounding
            assert float(np.abs(host(got)).max()) <= 1e-4, name
            continue
        _grad_close(host(got), w, "f32", name)

"""bf16 attention on each query block size that more than 128 keys can take (512, 256
and 128 queries per work-group, chosen by the number of work-groups), with partial
blocks and key tiles, and the many-query tiling of at most 32 keys: forward, row
statistics and gradients against the fp64 oracle at the bf16 bar."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_close, dev, host, say
from tests.test_gpu_attention_general import _grad_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,X,Lq,Lk,H,Hkv,D", [
    (1, 1, 129, 129, 2, 2, 72),     # 128: one full block and one query, a key past two tiles
    (1, 1, 300, 200, 2, 1, 64),     # 128
    (1, 1, 257, 130, 1, 1, 96),     # 128, widest head
    (2, 65, 130, 140, 2, 2, 72),    # 260 units of two 128 blocks or one 256 block
    (1, 40, 260, 150, 8, 8, 72),    # 320 units of 260 queries
    (1, 32, 520, 150, 8, 8, 32),    # 256 units of 520 queries
    (1, 2, 300, 20, 2, 2, 72), (1, 3, 256, 32, 2, 1, 80), (1, 2, 700, 1, 2, 2, 64),   # few keys, many queries
])
def test_query_blocks(B, X, Lq, Lk, H, Hkv, D):
    import paper_2403_10266_amd as dsp
    rng = np.random.default_rng(Lq + 3 * Lk + D)
    q = synth.bf16_round(rng.standard_normal((B, X, Lq, H * D), dtype=np.float32))
    k, v = (synth.bf16_round(rng.standard_normal((B, X, Lk, Hkv * D), dtype=np.float32)) for _ in range(2))
    do = synth.bf16_round(rng.standard_normal(q.shape, dtype=np.float32))
    say(f"query blocks B={B} X={X} Lq={Lq} Lk={Lk} H={H} Hkv={Hkv} D={D}")
    qd, kd, vd = (dev(a, "bf16") for a in (q, k, v))
    o, lse = dsp.dsp_attn_general(qd, kd, vd, H, Hkv, with_lse=True)
    assert_close(host(o), oracle.attention_grouped(q, k, v, H, Hkv), "bf16", "o")
    if Lk > 1 and B * X * Lq < 6000:
        grads = dsp.dsp_attn_general_bwd(qd, kd, vd, o, dev(do, "bf16"), lse, H, Hkv)
        for got, w, name in zip(grads, oracle.attention_grouped_bwd(q, k, v, do, H, Hkv), ("dq", "dk", "dv")):
            _grad_close(host(got), w, "bf16", name)


@pytest.mark.parametrize("B,X,Lq,Lk,H,Hkv,D", [
    (1, 2, 129, 257, 2, 2, 72),     # both kernels on 4 waves
    (1, 34, 400, 130, 16, 16, 16),  # 544 units of 400 queries (4 waves), 130 keys
    (1, 40, 256, 150, 16, 16, 16),  # 640 units of exactly one 8-wave query block
    (1, 7, 300, 140, 8, 2, 64),     # grouped heads: fewer dK/dV work-groups
])
def test_backward_waves(B, X, Lq, Lk, H, Hkv, D):
    import paper_2403_10266_amd as dsp
    rng = np.random.default_rng(Lq + 3 * Lk + D)
    q, do = (synth.bf16_round(rng.standard_normal((B, X, Lq, H * D), dtype=np.float32)) for _ in range(2))
    k, v = (synth.bf16_round(rng.standard_normal((B, X, Lk, Hkv * D), dtype=np.float32)) for _ in range(2))
    say(f"backward waves B={B} X={X} Lq={Lq} Lk={Lk} H={H} Hkv={Hkv} D={D}")
    qd, kd, vd = (dev(a, "bf16") for a in (q, k, v))
    o, lse = dsp.dsp_attn_general(qd, kd, vd, H, Hkv, with_lse=True)
    grads = dsp.dsp_attn_general_bwd(qd, kd, vd, o, dev(do, "bf16"), lse, H, Hkv)
    for got, w, name in zip(grads, oracle.attention_grouped_bwd(q, k, v, do, H, Hkv), ("dq", "dk", "dv")):
        _grad_close(host(got), w, "bf16", name)

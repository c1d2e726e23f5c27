"""bf16 attention on each query block size that more than 128 keys can take (512, 256
and 128 queries per work-group, chosen by the number of work-groups), with partial
blocks and key tiles, and the many-query tiling of at most 32 keys: forward, row
statistics and gradients against the fp64 oracle at the bf16 bar; the gradients'
kernels with four and with eight waves per work-group.  Each case names the variants
it means and asserts that the launch takes them.  Frames are independent, so where
there are many the first and the last are compared."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_close, dev, host, say
from tests.test_gpu_attention_general import _grad_close
from tests.test_gpu_attention_range import D as RAMP_D, H as RAMP_H, late_moves, ramp_inputs
from tests.test_launch_choices_cpu import attn_bwd, attn_fwd

pytestmark = pytest.mark.gpu


def _frames(X):
    return [0] if X == 1 else [0, X - 1]


def _lse(q, k, H, Hkv):
    """log-sum-exp of the scaled scores, (B, X, H, Lq), float64"""
    B, X, Lq, C = q.shape
    D = C // H
    q = q.astype(np.float64).reshape(B, X, Lq, H, D)
    k = np.repeat(k.astype(np.float64).reshape(B, X, -1, Hkv, D), H // Hkv, axis=3)
    s = np.einsum("bxqhd,bxkhd->bxhqk", q, k, optimize=True) / np.sqrt(D)
    m = s.max(-1, keepdims=True)
    return (m + np.log(np.exp(s - m).sum(-1, keepdims=True)))[..., 0]


def _check(got_o, got_lse, q, k, v, H, Hkv):
    at = _frames(q.shape[1])
    qs, ks, vs = (t[:, at] for t in (q, k, v))
    assert_close(host(got_o)[:, at], oracle.attention_grouped(qs, ks, vs, H, Hkv), "bf16", "o")
    # Q' is rounded to bf16 before the products: a score is off by at most 2^-9 sum |q| |k| / sqrt(D)
    D = q.shape[3] // H
    mag = np.abs(qs).max() * np.abs(ks).reshape(*ks.shape[:3], Hkv, D).sum(-1).max() / np.sqrt(D)
    err = np.abs(host(got_lse)[:, at] - _lse(qs, ks, H, Hkv)).max()
    say(f"  lse: max_abs={err:.3e} (bound {2.0 ** -9 * mag:.3e})")
    assert err <= 2.0 ** -9 * mag


def _check_grads(dsp, o, lse, qd, kd, vd, q, k, v, do, H, Hkv):
    at = _frames(q.shape[1])
    grads = dsp.dsp_attn_general_bwd(qd, kd, vd, o, dev(do, "bf16"), lse, H, Hkv)
    want = oracle.attention_grouped_bwd(*(t[:, at] for t in (q, k, v, do)), H, Hkv)
    for got, w, name in zip(grads, want, ("dq", "dk", "dv")):
        _grad_close(host(got)[:, at], w, "bf16", name)


@pytest.mark.parametrize("B,X,Lq,Lk,H,Hkv,D,queries", [
    (1, 1, 129, 129, 2, 2, 72, 128),     # one full block and one query, a key past two tiles
    (1, 1, 300, 200, 2, 1, 64, 128),
    (1, 1, 257, 130, 1, 1, 96, 128),     # widest head
    (2, 65, 130, 140, 2, 2, 72, 128),    # 260 units of two blocks
    (1, 40, 260, 150, 8, 8, 72, 128),    # 320 units of 260 queries
    (1, 32, 520, 150, 8, 8, 32, 128),    # 256 units of 520 queries
    (1, 16, 300, 130, 8, 8, 72, 256), (1, 16, 300, 200, 8, 4, 64, 256), (1, 60, 250, 250, 16, 16, 72, 256),
    (1, 32, 500, 321, 8, 8, 72, 512), (1, 32, 500, 700, 8, 2, 32, 512), (1, 32, 500, 321, 8, 8, 80, 512),
    (1, 16, 980, 1000, 8, 8, 72, 512),
    (1, 2, 300, 20, 2, 2, 72, 128), (1, 2, 700, 1, 2, 2, 64, 128), (1, 52, 1100, 17, 8, 4, 32, 128),   # few keys,
    (1, 20, 1030, 31, 8, 8, 80, 128),                                                                  # many queries
    (1, 3, 256, 32, 2, 1, 80, 32), (1, 3, 300, 30, 2, 2, 16, 32), (1, 2, 255, 32, 2, 2, 72, 32),       # few of both
])
def test_query_blocks(B, X, Lq, Lk, H, Hkv, D, queries):
    import paper_2403_10266_amd as dsp
    assert attn_fwd(D, B * X * H, Lq, Lk, H * D) == queries
    rng = np.random.default_rng(Lq + 3 * Lk + D)
    q = synth.bf16_round(rng.standard_normal((B, X, Lq, H * D), dtype=np.float32))
    k, v = (synth.bf16_round(rng.standard_normal((B, X, Lk, Hkv * D), dtype=np.float32)) for _ in range(2))
    do = synth.bf16_round(rng.standard_normal(q.shape, dtype=np.float32))
    say(f"query blocks B={B} X={X} Lq={Lq} Lk={Lk} H={H} Hkv={Hkv} D={D}")
    qd, kd, vd = (dev(a, "bf16") for a in (q, k, v))
    o, lse = dsp.dsp_attn_general(qd, kd, vd, H, Hkv, with_lse=True)
    _check(o, lse, q, k, v, H, Hkv)
    if Lk > 1:
        _check_grads(dsp, o, lse, qd, kd, vd, q, k, v, do, H, Hkv)


@pytest.mark.parametrize("X,L,queries", [(64, 300, 256), (128, 500, 512), (2, 300, 128)])
def test_query_blocks_moved_reference(X, L, queries):
    """Later key tiles hold larger scores, so the running reference moves on the way."""
    import paper_2403_10266_amd as dsp
    H, D = RAMP_H, RAMP_D
    assert attn_fwd(D, X * H, L, L, H * D) == queries
    q, k, v, _ = ramp_inputs(L, "bf16", seed=600 + L, X=X)
    at = _frames(X)
    moves = late_moves(q[:, at], k[:, at], D ** -0.5)
    say(f"query blocks, moved reference X={X} L={L}: {moves} late moves in the compared frames")
    assert moves > 0
    o = dsp.dsp_attn_general(*(dev(a, "bf16") for a in (q, k, v)), H, H)
    assert_close(host(o)[:, at], oracle.attention_grouped(q[:, at], k[:, at], v[:, at], H, H), "bf16", "o")


@pytest.mark.parametrize("B,X,Lq,Lk,H,Hkv,D,waves", [
    (1, 2, 129, 257, 2, 2, 72, (4, 4)),
    (1, 34, 400, 130, 16, 16, 16, (4, 4)),   # 544 units of 400 queries, 130 keys
    (1, 40, 256, 150, 16, 16, 16, (4, 4)),   # 640 units of exactly one block of 256 queries
    (1, 7, 300, 140, 8, 2, 64, (4, 4)),      # grouped heads: fewer dK/dV work-groups
    (1, 8, 400, 130, 16, 16, 72, (8, 4)), (1, 14, 250, 300, 16, 4, 64, (8, 4)), (1, 32, 250, 140, 8, 4, 96, (8, 4)),
    (1, 24, 1000, 130, 8, 8, 72, (4, 8)),
    (1, 16, 250, 250, 16, 16, 72, (8, 8)), (1, 32, 250, 140, 8, 8, 80, (8, 8)), (1, 30, 255, 250, 8, 8, 72, (8, 8)),
    (1, 3, 100, 70, 4, 2, 72, (4, 4)),       # up to 128 positions, few work-groups: two key tiles at once
    (1, 140, 100, 70, 4, 2, 64, (4, 4)),     # more of them: one at a time
])
def test_backward_waves(B, X, Lq, Lk, H, Hkv, D, waves):
    import paper_2403_10266_amd as dsp
    assert attn_bwd(D, B * X, H, Hkv, Lq, Lk) == waves
    rng = np.random.default_rng(Lq + 3 * Lk + D)
    q, do = (synth.bf16_round(rng.standard_normal((B, X, Lq, H * D), dtype=np.float32)) for _ in range(2))
    k, v = (synth.bf16_round(rng.standard_normal((B, X, Lk, Hkv * D), dtype=np.float32)) for _ in range(2))
    say(f"backward waves B={B} X={X} Lq={Lq} Lk={Lk} H={H} Hkv={Hkv} D={D}")
    qd, kd, vd = (dev(a, "bf16") for a in (q, k, v))
    o, lse = dsp.dsp_attn_general(qd, kd, vd, H, Hkv, with_lse=True)
    _check_grads(dsp, o, lse, qd, kd, vd, q, k, v, do, H, Hkv)

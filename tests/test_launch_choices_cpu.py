"""The variants that launches choose, asked without a device: a choice has to be one
that can be launched wherever another variant can (a grid dimension takes fewer than
2^32 threads), and the variants that the GPU tests name are the ones they run."""
import ctypes

import pytest

import paper_2403_10266_amd as dsp

I64, INT = ctypes.c_int64, ctypes.c_int
GRID_THREADS = 1 << 32


def attn_fwd(D, units, L, Lk, stride=1152):
    f = dsp.lib().dsp_choice_attn_fwd
    f.restype, f.argtypes = INT, [INT, I64, I64, I64, I64]
    return f(D, units, L, Lk, stride)


# threads of a work-group by its queries, for more than 128 keys and for at most 32
ATTN_THREADS = {"many": {512: 512, 256: 256, 128: 256}, "few": {128: 256, 32: 64}}


@pytest.mark.parametrize("L", [256, 257, 300, 512, 1000, 4096])
@pytest.mark.parametrize("Lk", [1, 20, 32, 129, 300, 1000])
@pytest.mark.parametrize("D", [16, 72])
def test_attention_forward_grid(L, Lk, D):
    kind = "few" if Lk <= 32 else "many"
    threads, base = ATTN_THREADS[kind], 32 if Lk <= 32 else 512
    most = (GRID_THREADS - 1) // (-(-L // base) * threads[base])    # units that blocks of `base` queries can launch
    for units in (most, most - 1, most * 3 // 4, most // 2 + 1, most // 2):
        q = attn_fwd(D, units, L, Lk)
        assert units * -(-L // q) * threads[q] < GRID_THREADS, (units, q)


@pytest.mark.parametrize("D,units,L,queries", [
    (16, 2048, 4096, 32), (32, 512, 257, 32), (32, 512, 1023, 32), (32, 128, 1024, 32), (32, 256, 1024, 128),
    (64, 1, 256, 128), (72, 4, 257, 128), (72, 4, 255, 32), (80, 64, 1024, 32), (80, 128, 1024, 128), (96, 128, 257, 32),
    (96, 512, 257, 128),
])
def test_attention_forward_few_keys(D, units, L, queries):
    assert attn_fwd(D, units, L, 20) == queries


def test_attention_forward_widest_head():
    """At D = 96 the 256-query instance spills registers: never chosen."""
    for units in (4, 32, 128, 512, 2048):
        for L, Lk in ((150, 150), (300, 300), (512, 129), (1024, 300), (2000, 500)):
            assert attn_fwd(96, units, L, Lk) != 256
    assert attn_fwd(72, 512, 2000, 500) == 256


def attn_bwd(D, bx, H, Hkv, L, Lk):
    """(waves of dQ, waves of dK/dV) per work-group"""
    f = dsp.lib().dsp_choice_attn_bwd
    f.restype, f.argtypes = INT, [INT, I64, INT, INT, I64, I64]
    v = f(D, bx, H, Hkv, L, Lk)
    return v & 255, v >> 8


def test_attention_backward_waves_near_ties():
    """Four and eight waves within a few percent of each other: four only at the head
    widths, and over the tiles, where three of their work-groups share a CU."""
    assert attn_bwd(80, 128, 4, 4, 150, 150) == (8, 8)
    assert attn_bwd(80, 512, 4, 4, 1024, 1024) == (8, 8)
    assert attn_bwd(32, 128, 4, 4, 150, 150) == (8, 8)
    assert attn_bwd(72, 128, 4, 4, 150, 150) == (4, 8)
    assert attn_bwd(72, 512, 4, 4, 1024, 1024) == (4, 8)


def linear(M, N, K, gelu=False):
    """(rows, columns, whether four K slices are in flight) of the output tile"""
    f = dsp.lib().dsp_choice_linear
    f.restype, f.argtypes = ctypes.c_uint32, [I64, I64, I64, INT]
    v = f(M, N, K, gelu)
    return (v >> 16) & 0x7FFF, v & 0xFFFF, bool(v >> 31)


def weight_grad(M, N, K):
    """((rows, columns, whether four slices are in flight) of the output tile, splits)"""
    f = dsp.lib().dsp_choice_weight_grad
    splits = INT()
    f.restype, f.argtypes = ctypes.c_uint32, [I64, I64, I64, ctypes.POINTER(INT)]
    v = f(M, N, K, ctypes.byref(splits))
    return ((v >> 16) & 0x7FFF, v & 0xFFFF, bool(v >> 31)), splits.value


def test_weight_gradient_workspace():
    """No workspace, and no split, up to 3968 tokens; at most what the workspace holds past it."""
    ws = dsp.lib().dsp_linear_bwd_weight_workspace_bytes
    for N, K in ((1152, 1152), (576, 4608), (8, 8)):
        assert ws(3968, N, K, dsp.DSP_BF16) == 0 and weight_grad(3968, N, K)[1] == 1
    assert ws(3969, 1152, 1152, dsp.DSP_BF16) > 0
    for M in (3969, 5001, 13600, 32768):
        for N, K in ((1152, 1152), (3456, 1152), (1152, 4608), (640, 72)):
            need = ws(M, N, K, dsp.DSP_BF16)
            assert weight_grad(M, N, K)[1] <= max(1, need // (4 * N * K))


@pytest.mark.parametrize("N", [8, 64, 136, 1152])
@pytest.mark.parametrize("K", [64, 1024])
def test_linear_grid(N, K):
    # launches that 256-row tiles (256 threads) can make
    most = (GRID_THREADS // 256 - 1) // -(-N // 192) * 256
    for M in (1 << 20, 1 << 24, 1 << 28, (1 << 30) - 64, 1 << 30, (1 << 30) + 64, 3 << 29, (1 << 31) - 256):
        if M <= most:
            rows, cols, _ = linear(M, N, K)
            assert -(-M // rows) * -(-N // cols) * 256 < GRID_THREADS, (M, rows, cols)

"""The Python binding's checks: a tensor whose device, dtype, shape or layout
does not match what the C entry point reads and writes in place raises before
anything is launched (never copied behind the caller's back), and work passed
an explicit stream runs there, with its outputs allocated on it."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import bits16, dev, host, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.fixture(scope="module")
def dsp():
    import paper_2403_10266_amd as dsp
    return dsp


def test_switch_rejects_views_and_bad_out(torch, dsp):
    x = torch.zeros((1, 8, 16, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError, match="contiguous"):
        dsp.dsp_switch(x.transpose(1, 2), 1, 2, 2)
    with pytest.raises(ValueError, match="dtype|must be"):
        dsp.dsp_switch(x, 1, 2, 2, out=torch.empty(x.shape, dtype=torch.float32, device="cuda"))
    with pytest.raises(ValueError, match="elements"):
        dsp.dsp_switch(x, 1, 2, 2, out=torch.empty(x.numel() // 2, dtype=torch.bfloat16, device="cuda"))
    with pytest.raises(ValueError, match="device"):
        dsp.dsp_switch(x.cpu(), 1, 2, 2)


def test_attention_rejects_mismatched_layouts(torch, dsp):
    B, T, S, H, D = 1, 2, 40, 2, 72
    C = H * D
    qkv = torch.zeros((B, T, S, 3 * C), dtype=torch.bfloat16, device="cuda")
    q = qkv[..., :C]
    k = torch.zeros((B, T, S, C), dtype=torch.bfloat16, device="cuda")   # dense: row stride C, not 3C
    with pytest.raises(ValueError, match="row stride"):
        dsp.dsp_spatial_attn(q, k, qkv[..., 2 * C:], H, C=C)
    with pytest.raises(ValueError, match="must be"):
        dsp.dsp_spatial_attn(k, k.float(), k, H)
    with pytest.raises(ValueError):
        dsp.dsp_spatial_attn(k, k, k, H, out=torch.empty((B, T, S - 1, C), dtype=torch.bfloat16, device="cuda"))
    with pytest.raises(ValueError):
        dsp.dsp_attn_strided(k, k, k.transpose(1, 2).contiguous().transpose(1, 2), H)


def test_linear_and_block_reject_bad_tensors(torch, dsp):
    a = torch.zeros((64, 128), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((32, 128), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError, match="contiguous"):
        dsp.dsp_linear(a.t().contiguous().t(), w)
    with pytest.raises(ValueError, match="w must be"):
        dsp.dsp_linear(a, w[:, :64].contiguous())
    with pytest.raises(ValueError, match="residual"):
        dsp.dsp_linear(a, w, residual=torch.zeros((64, 32), dtype=torch.bfloat16, device="cuda"),
                       epilogue=dsp.DSP_EPI_RESID)
    B, T, S, C, H = 1, 2, 8, 64, 4
    x = torch.zeros((B, T, S, C), dtype=torch.float32, device="cuda")
    wts = {"wqkv_s": torch.zeros((3 * C, C), dtype=torch.float32, device="cuda"),
           "wo_s": torch.zeros((C, C), dtype=torch.float32, device="cuda"),
           "wqkv_t": torch.zeros((3 * C, C), dtype=torch.float32, device="cuda"),
           "wo_t": torch.zeros((C, C), dtype=torch.float32, device="cuda")}
    with pytest.raises(ValueError, match="must be"):
        dsp.dsp_st_block_forward(x.to(torch.bfloat16), wts, H, flags=dsp.DSP_BLOCK_ATTN_ONLY)
    bad = dict(wts, wo_t=torch.zeros((C, C + 8), dtype=torch.float32, device="cuda"))
    with pytest.raises(ValueError, match="wo_t"):
        dsp.dsp_st_block_forward(x, bad, H, flags=dsp.DSP_BLOCK_ATTN_ONLY)
    with pytest.raises(ValueError, match="w1"):
        dsp.dsp_st_block_forward(x, wts, H)                 # the MLP needs w1 and w2


def test_explicit_stream(torch, dsp):
    """The switch and an attention call on a side stream: same bits as on the
    current stream, outputs allocated on the side stream."""
    rng = np.random.default_rng(3)
    x = synth.bf16_round(rng.standard_normal((2, 16, 32, 144), dtype=np.float32))
    xd = dev(x, "bf16")
    base = dsp.dsp_switch(xd, 1, 2, 4)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    y = dsp.dsp_switch(xd, 1, 2, 4, stream=side)
    q, k, v = (dev(synth.bf16_round(rng.standard_normal((1, 2, 100, 144), dtype=np.float32)), "bf16")
               for _ in range(3))
    o = dsp.dsp_spatial_attn(q, k, v, 2, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert np.array_equal(bits16(y), bits16(base))
    want = oracle.spatial_attention(*(host(t) for t in (q, k, v)), 2)
    assert_close(host(o), want, "bf16", "attention on a side stream")


def test_current_stream_without_the_internal_handle(torch, dsp, monkeypatch):
    """Without torch's internal function for the raw handle, calls still run on the
    current stream: captured there, the launch is replayed."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    x = torch.arange(2 * 4 * 8 * 8, device="cuda").to(torch.float32).view(2, 4, 8, 8)
    y = torch.empty_like(x).view(-1)
    dsp.dsp_switch(x, 1, 2, 1, out=y)
    want = y.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dsp.dsp_switch(x, 1, 2, 1, out=y)
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)

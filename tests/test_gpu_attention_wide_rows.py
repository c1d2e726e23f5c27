"""bf16 cross-attention over few keys whose query rows lie far apart (queries along T
of a (B, T, S, C) tensor): a block of 128 such rows is past the 32-bit offsets of a
work-group, a block of 32 is not.  The results are those of packed queries."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride,Lq", [
    (1 << 23, 256),            # the smallest stride past a block of 128 rows
    ((1 << 25) - 8, 70),       # few queries: blocks of 32 at any stride
])
def test_wide_query_rows(stride, Lq):
    import torch

    import paper_2403_10266_amd as dsp
    H, D, Lk = 2, 72, 20
    gen = torch.Generator(device="cuda:0").manual_seed(Lq)
    q, k, v = (torch.randn((1, 1, n, H * D), generator=gen, device="cuda:0").to(torch.bfloat16) for n in (Lq, Lk, Lk))
    buf = torch.empty((Lq - 1) * stride + H * D, dtype=torch.bfloat16, device="cuda:0")
    wide = buf.as_strided(q.shape, (buf.numel(), buf.numel(), stride, 1))
    wide.copy_(q)
    say(f"wide query rows stride={stride} Lq={Lq}")
    got = dsp.dsp_attn_general(wide, k, v, H, H)
    assert torch.equal(got, dsp.dsp_attn_general(q, k, v, H, H))

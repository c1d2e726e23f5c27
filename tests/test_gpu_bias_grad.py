"""The bias gradient (column sums of dy) at the edges of its work-groups' row
steps and column groups, against float64 sums.

Bound: a column's sum is a chain of at most ceil(M / 64) fp32 adds per thread (1024
threads over at least 2, at most 16 threads per row), then 6 lane and 16 wave
adds, each rounding a partial sum no larger than the column's sum of
magnitudes: |error| <= (M / 64 + 23) 2^-24 sum |dy|."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, say
from tests.test_gpu_linear_bwd import _draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", [(1, 8), (8, 1160), (9, 1160), (16, 4104), (17, 40), (63, 24), (64, 16), (257, 40), (512, 1152), (2047, 1160), (2049, 128),
                                 (4100, 4096), (5000, 4104)])
def test_bias_gradient(dtype, M, N):
    import paper_2403_10266_amd as dsp
    dy, x = _draw((M, N), dtype, M + N), _draw((M, 8), dtype, 3)
    say(f"bias gradient {dtype} M={M} N={N}")
    _, db = dsp.dsp_linear_bwd_weight(dev(dy, dtype), dev(x, dtype), with_bias=True)
    d64 = dy.astype(np.float64)
    bound = (M / 64 + 23) * 2.0 ** -24 * np.abs(d64).sum(0)
    assert (np.abs(host(db) - d64.sum(0)) <= bound).all()

"""oda_argmax at the edges of its groups, threads and rounds: rows of one group
to several rounds of loads, equal maxima in other lanes, wavefronts and rounds
(the first wins), NaNs, infinities, rows of -infinity and NaN only."""
import numpy as np
import pytest
import torch

import oda_synth as S
from harness import dev_f32, need_gpu
from oracle import decoder as OD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 8, 4092, 16384, 16388, 32768, 32772, 65536, 65540, 151936])
def test_argmax_edges(n):
    P = need_gpu()
    g = S.rng(n, S.STREAM_DECODER)
    x = g.standard_normal((12, n)).astype(np.float32)
    last = n - 1
    x[1, [0, last]] = 50.0                                   # equal maxima, far apart
    x[2, last] = 50.0
    x[3, g.integers(0, n, 4)] = 50.0
    x[4, g.random(n) < 0.5] = np.nan
    x[5] = np.nan
    x[6] = -np.inf
    x[7] = -np.inf
    x[7, :last] = np.nan                                     # one -inf among NaNs
    x[8] = np.nan
    x[8, n // 2] = -3.0
    x[9, n // 3] = np.inf
    x[10] = np.float32(-3.4e38)
    x[11, 3::4] = 60.0                                       # every group's last value
    idx = torch.full((12,), 77, dtype=torch.int32, device="cuda")
    P.argmax(12, n, dev_f32(x), idx)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(idx.cpu().numpy(), OD.argmax(x))

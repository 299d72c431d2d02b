"""The split merge where whole splits weigh nothing: finite bf16 queries and keys
whose products overflow to -infinity in fp32 over ranges of positions as long
as those the merge's threads take (and over every cached position), with and
without a candidate, with fixed and automatic splits, against the fp64 oracle
(there the logits are finite and so low that the weights are zero).

Tolerance as everywhere against the oracle: 1e-4 absolute."""
import numpy as np
import pytest
import torch

import oda_synth as S
from harness import LSE_ABS, AttnProblem, check_close

pytestmark = pytest.mark.gpu

N = 1200


def _problem(lo, hi, cur, split_blocks, D):
    """Positions [lo, hi) have logits of -infinity, the others are as drawn with dimension 0 left out."""
    p = AttnProblem(11 + lo + D, 1, 2, 4, 2, D, np.array([N, 700], np.int32), cur=cur, split_blocks=split_blocks)
    huge, low = (S.f32_to_bf16_bits(np.float32(v)).item() for v in (3e38, -3e38))
    p.q[..., 0] = huge
    p.k[:, :, :, 0, :, 0] = 0                            # [L][block][Hkv][D / 8][16][8]
    if cur:
        p.kc[..., 0] = 0
    for pos in range(lo, hi):
        p.k[:, p.table[0, pos // 16], :, 0, pos % 16, 0] = low
    p.upload()
    return p


@pytest.mark.parametrize("lo,hi", [(0, 416), (320, 720), (800, N), (0, 1199)])
@pytest.mark.parametrize("cur", [False, True])
@pytest.mark.parametrize("split_blocks,D", [(2, 64), (2, 128), (0, 128)])
def test_splits_that_weigh_nothing(lo, hi, cur, split_blocks, D):
    p = _problem(lo, hi, cur, split_blocks, D)
    for run, oracle in ((p.run_full, p.oracle_full), (lambda: p.run_local(4, 1100), lambda: p.oracle_local(4, 1100))):
        out, lse = run()
        ro, rl = oracle()[:2]
        check_close(out.cpu().numpy(), ro, "out")
        assert np.abs(lse.cpu().numpy() - np.asarray(rl)).max() <= LSE_ABS


def test_nothing_to_attend_is_nan():
    """Every logit -infinity, the candidate's too: no weight, NaN rows, only for that request."""
    p = _problem(0, N, True, 2, 64)
    p.kc[0, 0, :, 0] = S.f32_to_bf16_bits(np.float32(-3e38)).item()
    p.upload()
    out = p.run_full()[0]
    assert bool(torch.isnan(out[:, 0]).all()) and bool(torch.isfinite(out[:, 1]).all())

"""The recall head for batches on the matrix-core tiles: request counts around
the vector kernels' limits, 8 and 16, tower widths around 8, 16 and the
32-element chunks, K shorter than a chunk and ragged over the wavefronts and
halves, and nonfinite inputs staying in their request.

Tolerance: scores are held to 4e-6 of the score scale.  A layer's fp32 sums of
up to 8192 terms of random sign err by about 2e-7 of their size (chains of at
most four, 32 and four additions), and the five layers' errors add."""
import numpy as np
import pytest
import torch

import oda_synth as S
from test_gate_parity import Gate, _check

pytestmark = pytest.mark.gpu


CASES = [
    ("paper", 4, 4, 4), ("paper", 100, 64, 3), ("paper", 36, 12, 8), ("paper", 68, 20, 9), ("paper", 516, 36, 16), ("paper", 1028, 124, 17),
    ("paper", 2052, 260, 33), ("paper", 264, 1028, 4), ("paper", 4096, 132, 65), ("mlp", 4, 4, 5), ("mlp", 100, 28, 8),
    ("mlp", 1020, 2052, 6), ("mlp", 8192, 516, 17), ("mlp", 8192, 516, 7),
    ("mlp", 4100, 1026 * 2, 8),
    # a workgroup per row instead of tiles, and past its limits
    ("mlp", 4096, 36, 5), ("mlp", 4100, 516, 5), ("mlp", 4096, 512, 6), ("mlp", 8196, 436, 7), ("mlp", 4096, 516, 6),
    ("mlp", 4100, 440, 7), ("mlp", 4092, 64, 7), ("mlp", 6148, 68, 8), ("mlp", 6144, 132, 17), ("mlp", 8196, 256, 16),
    # tiles of sixteen rows and requests
    ("paper", 516, 632, 70), ("paper", 1028, 1028, 40), ("mlp", 260, 1028, 70), ("mlp", 4100, 1028, 40)]


def test_both_tile_edges_are_among_the_cases():
    """Eight rows and requests up to 512 workgroups of them, else sixteen, for every layer of either head."""
    seen = set()
    for kind, _, dh, B in CASES:
        tall = B > (3 if kind == "paper" else 4)
        for layer, rows in (("tower", 3 * -(-dh // 8)), ("fusion", -(-dh // 8)), ("gate/up", -(-2 * dh // 8)),
                            ("down", -(-dh // 8))) if kind == "paper" else (("mlp", -(-dh // 8)),):
            if tall:
                seen.add((layer, rows * -(-B // 8) <= 512))
    assert len(seen) == 10


@pytest.mark.parametrize("kind,d,dh,B", CASES)
def test_tile_edges(kind, d, dh, B):
    gate = Gate(kind, d, dh, B, seed=d + dh)
    h, e, l = (x[0] for x in S.gate_inputs(d + B, 1, B, d))
    ref = gate.oracle(h.astype(np.float64), e.astype(np.float64), l.astype(np.float64))
    sc, _, _ = _check(gate, h, e, l, float(np.median(ref)) + 0.01)
    assert np.abs(sc - ref).max() <= 4e-6 * max(1.0, float(np.abs(ref).max()))


@pytest.mark.parametrize("kind,B", [("paper", 5), ("paper", 18), ("mlp", 9)])
def test_nonfinite_inputs_stay_in_their_request(kind, B):
    d, dh = 264, 40
    gate = Gate(kind, d, dh, B)
    h, e, l = (x[0].copy() for x in S.gate_inputs(3, 1, B, d))
    clean = gate.run(h, e, l, 1e9)[0]
    l[1, 7] = np.nan
    l[2, 100] = np.inf
    sc, fl, wl, n = gate.run(h, e, l, 1e9)
    assert not np.isfinite(sc[1]) and fl[1] == 1
    assert kind == "mlp" or (not np.isfinite(sc[2]) and fl[2] == 1)   # inf / inf in the norm
    keep = [b for b in range(B) if b not in (1, 2)]
    assert np.array_equal(sc[keep], clean[keep]) and not fl[keep].any()


@pytest.mark.parametrize("d,dh,B", [(100, 28, 9), (1056, 32, 5), (1060, 2100, 70)])
def test_an_infinite_weight_gives_an_infinite_score(d, dh, B):
    """In the row's first elements too, which the chunk padding reads again."""
    gate = Gate("mlp", d, dh, B, seed=d)
    gate.params[0] = np.inf                               # W1[0][0]
    gate.params[dh * d + dh] = 0.5                        # w2[0]
    gate.dparams.copy_(torch.from_numpy(gate.params))
    h, e, l = (x[0].copy() for x in S.gate_inputs(3, 1, B, d))
    l[:, 0] = 1.0
    sc, fl, _, _ = gate.run(h, e, l, 1e9)
    assert np.all(sc == np.inf) and fl.all()

"""oda_dense_bf16 for several requests at the edges of its tiles: row counts
around 8, 16 and 32, request counts around 8, 16 and 32, K around the 32-element
steps, the 64-element chunks and the eight wavefronts' stretches, selection
lists with ids outside the batch, and nonfinite inputs, against the fp64 oracle.

Tolerance.  Every product is exact (bf16 weights, inputs as three bf16 pieces)
and an output is a chain of at most 32 additions in an instruction, K / 256
instructions per wavefront, 8 wavefronts, the low-piece sum and the epilogue,
all in fp32: |err| <= n 2^-24 sum_k |w x'| with n = K / 256 + 64 (plus the
rounding of the normalised input, 4 units).
"""
import numpy as np
import pytest
import torch

import oda_synth as S
from harness import dev_f32, dev_i32, dev_u16, need_gpu
from oracle import attention as OA
from oracle import decoder as OD

pytestmark = pytest.mark.gpu


def _bound(W, xn, K):
    """Per-output error bound of y = W x' ([B][rows])."""
    return (K / 256 + 68) * 2.0 ** -24 * (np.abs(xn) @ np.abs(OA.bf16_to_f64(W)).T)


def _inputs(seed, K, rows, B):
    g = S.rng(seed, S.STREAM_DECODER)
    W = S.normal_bf16(g, (rows, K), K ** -0.5)
    x = (g.standard_normal((B, K)) * np.exp(4 * g.standard_normal((B, 1)))).astype(np.float32)
    return g, W, x


PLAIN = [(1, 2), (8, 8), (17, 9), (33, 16), (2050, 3), (2056, 17), (4112, 33), (8208, 7), (2048, 32), (2041, 31)]
SWIGLU = [(8, 5, 2), (72, 17, 8), (520, 2056, 4), (1000, 4104, 16), (2048, 6152, 3), (264, 6160, 33), (264, 6144, 8),
          (520, 6137, 7), (136, 4096, 16), (1000, 4089, 15)]


def _tile(swiglu, N, B):
    """Row tiles and tile edge of the launch: the narrowest with one workgroup per CU at most, else the widest."""
    shapes = [(1, 8), (2, 8)] + ([(3, 8)] if swiglu else []) + [(1, 16), (2, 16)] + ([(3, 16)] if swiglu else [])
    return next((t for t in shapes if -(-N // (t[0] * t[1])) * -(-B // t[1]) <= 256), shapes[-1])


def test_every_tile_shape_is_among_the_cases():
    assert {_tile(False, N, B) for N, B in PLAIN} == {(1, 8), (2, 8), (1, 16), (2, 16)}
    assert {_tile(True, N, B) for _, N, B in SWIGLU} == {(p, e) for p in (1, 2, 3) for e in (8, 16)}


@pytest.mark.parametrize("K", [8, 40, 264, 1000, 2088])
@pytest.mark.parametrize("N,B", PLAIN)
def test_plain_tiles(K, N, B):
    P = need_gpu()
    g, W, x = _inputs(K * 7 + N + B, K, N, B)
    norm, residual = (N + B) % 2 == 0, B % 3 != 0
    gain = (1 + 0.02 * g.standard_normal(K)).astype(np.float32) if norm else None
    r = g.standard_normal((B, N)).astype(np.float32) if residual else None
    y = torch.full((B, N), np.nan, device="cuda")
    P.dense_bf16(P.dense_desc(K, N, P.DENSE_PLAIN, dev_u16(W), dev_f32(gain) if norm else None, 1e-6), B, dev_f32(x),
                 dev_f32(r) if residual else None, y)
    torch.cuda.synchronize()
    xn = OD.rmsnorm(x.astype(np.float64), gain, 1e-6) if norm else x.astype(np.float64)
    ref = OD.dense(W, x, gain, 1e-6, r)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= _bound(W, xn, K) + 2.0 ** -23 * np.abs(ref))


@pytest.mark.parametrize("K,N,B", SWIGLU)
def test_swiglu_tiles_with_a_list(K, N, B):
    P = need_gpu()
    g, W, x = _inputs(K + N + B, K, 2 * N, B)
    gain = (1 + 0.02 * g.standard_normal(K)).astype(np.float32)
    sel = [b for b in range(B) if b % 3 != 1][::-1]
    listed = sel[:1] + [B + 5] + sel[1:] + [-2]          # ids outside the batch are skipped
    listed = listed[:B]
    done = [b for b in listed if 0 <= b < B]
    y = torch.full((B, N), 7.0, device="cuda")
    P.dense_bf16(P.dense_desc(K, N, P.DENSE_SWIGLU, dev_u16(W), dev_f32(gain), 1e-6), B, dev_f32(x), None, y,
                 dev_i32(listed + [0] * (B - len(listed))), dev_i32([len(listed)]))
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    xn = OD.rmsnorm(x[done].astype(np.float64), gain, 1e-6)
    bound = _bound(W, xn, K)
    w64 = OA.bf16_to_f64(W)
    gate, up = xn @ w64[:N].T, xn @ w64[N:].T
    # |SiLU'| <= 1.1, |SiLU(z)| <= |z|; the hardware exponential adds a few units of SiLU(z)
    tol = 1.1 * bound[:, :N] * np.abs(up) + np.abs(gate) * bound[:, N:] + 2.0 ** -20 * np.abs(gate * up) + 1e-30
    ref = OD.swiglu(W, x[done], gain, 1e-6)
    assert np.all(np.abs(got[done] - ref) <= tol)
    assert np.all(got[[b for b in range(B) if b not in done]] == 7.0)


@pytest.mark.parametrize("B", [2, 9])
def test_nonfinite_inputs_stay_in_their_request(B):
    """An infinity gives the infinities (or NaN) that a sum of its products
    gives, a NaN gives NaN, the largest finite values do not overflow in the
    split, and no other request changes."""
    P = need_gpu()
    K, N = 136, 40
    g, W, x = _inputs(B, K, N, B)
    W[:, 5] = S.f32_to_bf16_bits(np.where(np.arange(N) % 2 == 0, 0.5, -0.25).astype(np.float32))
    clean = torch.empty(B, N, device="cuda")
    desc = P.dense_desc(K, N, P.DENSE_PLAIN, dev_u16(W))
    P.dense_bf16(desc, B, dev_f32(x), None, clean)
    bad = x.copy()
    bad[0] = 0.0
    bad[0, 5] = np.inf
    bad[1, 7] = np.nan
    if B > 2:
        bad[2] = 0.0
        bad[2, 5] = np.finfo(np.float32).max
    y = torch.empty(B, N, device="cuda")
    P.dense_bf16(desc, B, dev_f32(bad), None, y)
    torch.cuda.synchronize()
    got, clean = y.cpu().numpy(), clean.cpu().numpy()
    assert np.array_equal(got[0], np.where(np.arange(N) % 2 == 0, np.inf, -np.inf).astype(np.float32))
    assert np.all(np.isnan(got[1]))
    if B > 2:
        big = np.finfo(np.float32).max
        assert np.array_equal(got[2], np.where(np.arange(N) % 2 == 0, np.float32(0.5) * big, np.float32(-0.25) * big))
    assert np.array_equal(got[3:], clean[3:])


@pytest.mark.parametrize("K,N,B", [(K, N, B) for K in (8, 136, 544, 1536) for N, B in ((24, 2), (24, 9), (5000, 17))]
                         + [(1536, 65552, 1)])
def test_infinite_weights_and_gains(K, N, B):
    """A row with an infinite weight gives the infinity (or NaN) that a sum of
    its products gives, wherever in K it lies (the stretch padding repeats a
    row's first elements), whatever the lower bf16 pieces of the inputs; an
    infinite gain alike; a NaN with only low payload bits stays a NaN."""
    P = need_gpu()
    g, W, x = _inputs(K + N + B, K, N, B)
    x = np.abs(x) + 0.5
    x[:, ::3] = 1.0                                        # its lower pieces are zero
    inf, ninf = (int(S.f32_to_bf16_bits(np.full(1, v, np.float32))[0]) for v in (np.inf, -np.inf))
    W[1, 0], W[2, K - 1], W[3, K // 2], W[4, 0], W[4, K - 2] = inf, ninf, inf, inf, ninf
    rows = {1: np.inf, 2: -np.inf, 3: np.inf, 4: np.nan}
    clean = np.setdiff1d(np.arange(N), list(rows))
    gain = np.ones(K, np.float32)

    def run(x, gain):
        y = torch.empty(B, N, device="cuda")
        P.dense_bf16(P.dense_desc(K, N, P.DENSE_PLAIN, dev_u16(W), dev_f32(gain) if gain is not None else None, 1e-6), B,
                     dev_f32(x), None, y)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    for y in (run(x, None), run(x, gain)):
        for r, v in rows.items():
            assert np.array_equal(y[:, r], np.full(B, v, np.float32), equal_nan=True), (r, y[:, r])
        assert np.all(np.isfinite(y[:, clean]))
    gain[K - 1] = np.inf
    want = np.where(OA.bf16_to_f64(W[:, K - 1]) > 0, np.inf, -np.inf)
    some = clean[OA.bf16_to_f64(W[clean, K - 1]) != 0]
    assert np.array_equal(run(x, gain)[:, some], np.tile(want[some], (B, 1)))
    x[B - 1, K - 1] = np.array([0x7f800001], np.uint32).view(np.float32)[0]
    y = run(x, None)
    assert np.all(np.isnan(y[B - 1])) and np.all(np.isfinite(y[:B - 1][:, clean]))


@pytest.mark.parametrize("K,N", [(512, 65512), (1536, 65504), (1536, 65505), (1544, 65512), (2048, 65533)])
def test_one_request_on_a_large_layer(K, N):
    """On the tiles from 65,505 rows and K = 1536 in steps of 512, else a wavefront per rows."""
    P = need_gpu()
    g, W, x = _inputs(K + N, K, N, 1)
    y = torch.empty(1, N, device="cuda")
    P.dense_bf16(P.dense_desc(K, N, P.DENSE_PLAIN, dev_u16(W)), 1, dev_f32(x), None, y)
    torch.cuda.synchronize()
    ref = OD.dense(W, x, None, 1e-6, None)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= _bound(W, x.astype(np.float64), K) + 2.0 ** -23 * np.abs(ref))

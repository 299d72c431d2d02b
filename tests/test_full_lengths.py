"""oda_full_decode_attn planned on the device from the selected requests'
lengths: the same call with a fixed split (the general path) and the fp64
oracle, over selections, batches around the wavefront's 64 lanes, lengths from
one position to many splits, lengths outside the range, listed ids outside the
batch and repeated calls on one workspace.

Tolerance: the two paths sum the same terms in other groups, fp32 sums of
softmax-weighted values of size ~1, P as two bf16 pieces (2^-16 of each term):
1e-4 absolute as for the oracle."""
import numpy as np
import pytest
import torch

import oda_synth as S
from harness import MAX_ABS_INTERNAL, AttnProblem, check_close, dev_i32, need_gpu

pytestmark = pytest.mark.gpu


def _lengths(kind, B, g):
    if kind == "ragged":
        return np.exp(g.uniform(np.log(1), np.log(3000), B)).astype(np.int32).clip(1, 3000)
    if kind == "one-long":
        n = np.full(B, 17, np.int32)
        n[B // 2] = 6000
        return n
    return np.full(B, 1024, np.int32)


@pytest.mark.parametrize("select", ["all", "flags", "list", "strange-list"])
@pytest.mark.parametrize("B,kind,L,D,cur", [(2, "one-long", 1, 128, True), (5, "ragged", 1, 128, False),
                                            (9, "equal", 3, 64, True), (33, "ragged", 1, 64, True),
                                            (64, "ragged", 1, 64, False), (70, "ragged", 1, 64, True)])
def test_plan_by_length_matches_fixed_splits(B, kind, L, D, cur, select):
    g = S.rng(B * 31 + L, S.STREAM_SEQ_LENS)
    seq = _lengths(kind, B, g)
    p = AttnProblem(B + L, L, B, 4, 2, D, seq, cur=cur, max_len=6016)
    chosen = sorted(g.permutation(B)[:max(1, B // 2)].tolist())
    sel = dict(all={}, flags=dict(flags=dev_i32([int(b in chosen) for b in range(B)])))
    sel["list"] = dict(work_list=dev_i32(chosen[::-1] + [0] * (B - len(chosen))), n_work=dev_i32([len(chosen)]))
    strange = (chosen[:1] + [B + 3, -1] + chosen[1:])[:B]
    sel["strange-list"] = dict(work_list=dev_i32(strange + [0] * (B - len(strange))), n_work=dev_i32([len(strange)]))
    done = list(range(B)) if select == "all" else [b for b in (strange if select == "strange-list" else chosen)
                                                   if 0 <= b < B]
    P = need_gpu()
    ws = torch.zeros(P.attn_workspace_size(p.shape, 0, 0), dtype=torch.uint8, device="cuda")
    outs = []
    for _ in range(3):                       # the same workspace: the tickets are left zero
        out, lse = p.new_out(3.0)
        k = sel[select]
        P.full_decode_attn(p.shape, p.inp, 0, k.get("flags"), k.get("work_list"), k.get("n_work"), out, lse, ws)
        torch.cuda.synchronize()
        outs.append((out.cpu().numpy(), lse.cpu().numpy()))
    assert all(np.array_equal(outs[0][i], o[i]) for o in outs for i in (0, 1))
    out, lse = outs[0]
    others = [b for b in range(B) if b not in done]
    assert np.all(out[:, others] == 3.0) and np.all(lse[:, others] == 3.0)
    p.shape.split_blocks = 64
    fout, flse = p.run_full(**sel[select])
    assert np.abs(out[:, done] - fout.cpu().numpy()[:, done]).max() <= MAX_ABS_INTERNAL
    assert np.abs(lse[:, done] - flse.cpu().numpy()[:, done]).max() <= MAX_ABS_INTERNAL
    few = sorted(done, key=lambda b: seq[b])
    few = sorted({few[0], few[len(few) // 2], few[-1]})
    ro, rl = p.oracle_full(requests=few)[:2]
    check_close(out[:, few], np.asarray(ro)[:, few], "out")
    assert np.abs(lse[:, few] - np.asarray(rl)[:, few]).max() <= MAX_ABS_INTERNAL


def test_lengths_outside_the_range_stay_in_their_request():
    """NaN rows for a zero, a negative and a too long length; the others as without them."""
    B = 6
    seq = np.array([700, 40, 1500, 33, 900, 5], np.int32)
    p = AttnProblem(3, 1, B, 4, 2, 64, seq, max_len=1504)
    bad = seq.copy()
    bad[[1, 3, 5]] = [0, -7, 1505]
    good = p.run_full()[0].cpu().numpy()
    p.dseq.copy_(dev_i32(bad))
    got = p.run_full()[0].cpu().numpy()
    assert np.all(np.isnan(got[:, [1, 3, 5]]))
    assert np.abs(got[:, [0, 2, 4]] - good[:, [0, 2, 4]]).max() <= MAX_ABS_INTERNAL


def test_an_empty_list_writes_nothing():
    p = AttnProblem(4, 1, 4, 4, 2, 64, np.array([700, 40, 1500, 33], np.int32))
    out, lse = p.new_out(9.0)
    p.run_full(work_list=dev_i32([0, 0, 0, 0]), n_work=dev_i32([0]), out=out, lse=lse)
    assert torch.all(out == 9.0) and torch.all(lse == 9.0)


def _aliased(seed, B, Hq, Hkv, D, seq, cur):
    """A problem over long histories whose logical blocks share 96 physical ones."""
    p = AttnProblem(seed, 1, B, Hq, Hkv, D, np.full(B, 16 * (96 // B), np.int32), cur=cur)
    p.seq = np.asarray(seq, np.int32)
    mb = -(-int(p.seq.max()) // 16)
    p.table = S.rng(seed, S.STREAM_TABLE).integers(0, p.nb, (B, mb)).astype(np.int32)
    p.shape = p.P.Shape(1, B, Hq, Hkv, D, mb, int(p.seq.max()), p.nb)
    p.upload()
    return p


# blocks x units: 17,764 in one round; 69,888 and 133,120 in two and more rounds; 590,000 from
# 1,024 blocks per CU, whose pairs are more than a list's grid holds
@pytest.mark.parametrize("B,Hq,Hkv,D,lo,hi", [(6, 4, 2, 128, 3622, 43790), (5, 16, 8, 128, 7000, 48921),
                                              (13, 20, 20, 64, 300, 16384), (8, 32, 32, 64, 8192, 65536)])
@pytest.mark.parametrize("select", ["all", "flags", "list"])
@pytest.mark.parametrize("cur", [False, True])
def test_long_histories(B, Hq, Hkv, D, lo, hi, select, cur):
    seq = [lo + (hi - lo) * i // (B - 1) for i in S.rng(B, S.STREAM_SEQ_LENS).permutation(B)]
    p = _aliased(B + D, B, Hq, Hkv, D, seq, cur)
    sel = dict(all={}, flags=dict(flags=dev_i32([1] * B)),
               list=dict(work_list=dev_i32(list(range(B))[::-1]), n_work=dev_i32([B])))[select]
    out, lse = (t.cpu().numpy() for t in p.run_full(**sel))
    again, _ = p.run_full(**sel)
    assert np.array_equal(out, again.cpu().numpy())
    p.shape.split_blocks = 128
    fout, flse = (t.cpu().numpy() for t in p.run_full(**sel))
    assert np.abs(out - fout).max() <= MAX_ABS_INTERNAL and np.abs(lse - flse).max() <= MAX_ABS_INTERNAL
    few = sorted({int(np.argmin(seq)), int(np.argmax(seq))}) if select == "all" else [int(np.argmin(seq))]
    ro, rl = p.oracle_full(requests=few)[:2]
    check_close(out[:, few], np.asarray(ro)[:, few], "out")
    assert np.abs(lse[:, few] - np.asarray(rl)[:, few]).max() <= MAX_ABS_INTERNAL

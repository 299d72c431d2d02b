"""The workloads whose speed is tracked on one MI355X, each one pass through
public entry points of paper_2609_20734_amd, as a decode server issues them.

Kinds of case (sizes from the repository's own workloads and benchmark, other
sizes of the same ranges by `draw`):

  attn     one attention call: Local or Full, one layer (how a model's layer
           loop calls it) or a stack, all requests or a work list, with the
           query and candidate given or built in the call from the QKV
           projection (the decoder's form)
  step     the attention step of a batch: Local from the rings over every
           layer, the recall head, Full over the flagged requests
  gate     the recall head alone: towers to flags and the compacted list
  mlp      a decoder layer's SwiGLU and down projections, all requests or the
           flagged ones (the Full retry)
  vocab    the vocabulary projection and the greedy token
  commit   the selected candidates of every layer into the paged cache and
           the rings
  decoder  a whole decode step of the Qwen3-1.7B-shaped decoder as a replayed
           graph: Local forward, recall head, (Full retry of the flagged
           requests,) logits, greedy token, commit

Lengths are spread evenly over a case's range and dealt to the requests by the
seed, so a case's work does not depend on the seed.  Values follow oda_synth's
distributions, drawn on the GPU.
"""
import math

import torch

import paper_2609_20734_amd as P
from paper_2609_20734_amd.decoder import Decoder, DecoderShape

BLOCK = 16
EPS = 1e-6
THETA = 1e6

_LLAMA = dict(Hq=32, Hkv=8, D=128)      # Llama-3-8B-shaped heads
_QWEN = dict(Hq=16, Hkv=8, D=128)       # Qwen3-1.7B-shaped heads


def listed():
    return [
        # one layer of a single request's Local forward in the decoder, the smallest call of every
        # step: query and candidate built in the call, 4 sinks and a 2,048-position window
        dict(name="attn-local-b1", kind="attn", branch="local", form="qkv", L=1, B=1, **_QWEN, lo=4139, hi=4139, sink=4,
             window=2048, listed=0),
        # one layer of a single request's Full forward at 32K positions
        dict(name="attn-full-b1", kind="attn", branch="full", form="cur", L=1, B=1, **_LLAMA, lo=32768, hi=32768, sink=0,
             window=0, listed=0),
        # one layer of the Full retry: 5 flagged of 32 ragged requests, 8K-64K positions
        dict(name="attn-full-listed", kind="attn", branch="full", form="cur", L=1, B=32, **_LLAMA, lo=8192, hi=65536,
             sink=0, window=0, listed=5),
        # the headline step of the Mixed batch (8 of its 32 layers): Local from the rings, the recall
        # head, Full over the 3 flagged requests of 32
        dict(name="step-mixed", kind="step", L=8, B=32, **_LLAMA, lo=8192, hi=65536, sink=4, window=2048, d=4096, dt=256,
             listed=3),
        # the recall head: one request (the Llama-shaped stack), the Mixed batch, the Hybrid batch
        dict(name="gate-b1", kind="gate", head="paper", d=4096, dt=256, B=1),
        dict(name="gate-b32", kind="gate", head="paper", d=4096, dt=256, B=32),
        dict(name="gate-b8-wide", kind="gate", head="paper", d=8192, dt=512, B=8),
        # a decoder layer's MLP for a batch of 32 requests
        dict(name="mlp-b32", kind="mlp", d=2048, F=6144, B=32, listed=0),
        # logits and greedy tokens of four requests
        dict(name="vocab-b4", kind="vocab", d=2048, V=151936, B=4),
        # the step's commit, Mixed batch: 32 layers, cache and rings
        dict(name="commit-b32", kind="commit", L=32, B=32, Hkv=8, D=128, lo=17, hi=700, sink=4, window=256),
        # a whole decode step of one request that stays Local, 31,400 tokens of context
        dict(name="decoder-b1", kind="decoder", L=28, d=2048, F=6144, V=151936, **_QWEN, dt=1024, B=1, lo=31400,
             hi=31400, sink=4, window=2048, listed=0),
        # a whole decode step of eight ragged requests, two of them retried with Full
        dict(name="decoder-b8", kind="decoder", L=28, d=2048, F=6144, V=151936, **_QWEN, dt=1024, B=8, lo=1537,
             hi=16001, sink=4, window=2048, listed=2),
    ]


def _log(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(v / multiple)) * multiple)


def _lengths_range(rng, lo, hi):
    a, b = _log(rng, lo, hi), _log(rng, lo, hi)
    return min(a, b), max(a, b)


def draw(rng):
    """One more case of the ranges above (heads, widths, batches, lengths, branches, forms)."""
    kind = rng.choice(["attn", "attn", "attn", "step", "gate", "gate", "mlp", "mlp", "vocab", "commit", "decoder"])
    hkv = rng.choice([2, 4, 8])
    heads = dict(Hq=hkv * rng.choice([1, 2, 4, 5, 8]), Hkv=hkv, D=rng.choice([64, 128, 128]))
    if kind == "attn":
        B = _log(rng, 1, 32)
        lo, hi = _lengths_range(rng, 200, 65536)
        branch = rng.choice(["local", "full"])
        form = rng.choice(["cur", "plain", "qkv"])
        c = dict(kind=kind, branch=branch, form=form, L=1 if form == "qkv" else rng.choice([1, 1, 2, 6]), B=B, **heads,
                 lo=lo, hi=hi, sink=0, window=0, listed=0)
        if branch == "local":
            c.update(sink=rng.choice([0, 4, 20]), window=_log(rng, 64, 4096))
        else:
            c.update(listed=rng.choice([0, 0, 1, max(1, B // 3)]), window=rng.choice([0, 0, 0, 4096]))
        return c
    if kind == "step":
        lo, hi = _lengths_range(rng, 1024, 65536)
        B = _log(rng, 1, 16)
        return dict(kind=kind, L=rng.randint(1, 8), B=B, **heads, lo=lo, hi=hi, sink=4, window=_log(rng, 128, 4096),
                    d=_log(rng, 512, 8192, 8), dt=_log(rng, 64, 512, 8), listed=rng.randint(0, max(1, B // 4)))
    if kind == "gate":
        return dict(kind=kind, head=rng.choice(["paper", "paper", "mlp"]), d=_log(rng, 512, 8192, 4),
                    dt=_log(rng, 64, 1024, 4), B=_log(rng, 1, 64))
    if kind == "mlp":
        B = _log(rng, 1, 64)
        return dict(kind=kind, d=_log(rng, 512, 4096, 8), F=_log(rng, 1024, 12288, 8), B=B,
                    listed=rng.choice([0, 0, max(1, B // 4)]))
    if kind == "vocab":
        return dict(kind=kind, d=_log(rng, 512, 4096, 8), V=_log(rng, 16000, 152000, 4), B=_log(rng, 1, 32))
    if kind == "commit":
        lo, hi = _lengths_range(rng, 1, 600)
        return dict(kind=kind, L=rng.randint(1, 32), B=_log(rng, 1, 32), Hkv=heads["Hkv"], D=heads["D"], lo=lo, hi=hi,
                    sink=4, window=_log(rng, 16, 256))
    lo, hi = _lengths_range(rng, 300, 16384)
    B = _log(rng, 1, 8)
    d = _log(rng, 512, 2048, 64)
    return dict(kind="decoder", L=rng.randint(2, 12), d=d, F=_log(rng, 1024, 6144, 64), V=_log(rng, 16000, 152000, 8),
                **heads, dt=_log(rng, 64, 1024, 8), B=B, lo=lo, hi=hi, sink=4, window=_log(rng, 128, 2048),
                listed=rng.randint(0, max(1, B // 3)))


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _lens(c):
    """The case's lengths, ascending: evenly spread over [lo, hi]."""
    B = c["B"]
    return [c["hi"] if B == 1 else c["lo"] + (c["hi"] - c["lo"]) * i // (B - 1) for i in range(B)]


def _flagged_ranks(c):
    """Which of the ascending lengths the flagged requests have (spread evenly), or all of them."""
    B, k = c["B"], min(c.get("listed", 0), c["B"])
    return [(2 * i + 1) * B // (2 * k) for i in range(k)]


def _local_count(n, sink, window):
    return min(n, min(sink, n) + min(window, n)) if sink + window < n else n


def _kv_bytes(c, counts):
    return float(sum(counts)) * c["L"] * c["Hkv"] * c["D"] * 4


def _attn_io(c, requests):
    """Query and candidate read, output and log-sum-exp written."""
    return float(requests) * c["L"] * (c["Hq"] * (c["D"] * 6 + 4) + 4 * c["Hkv"] * c["D"])


def _gate_params(head, d, dt):
    return P.gate_param_count(P.HEAD_PAPER if head == "paper" else P.HEAD_MLP, d, dt)


def _gate_work(head, d, dt, B):
    n = _gate_params(head, d, dt)
    return 4.0 * n + 4.0 * B * d * (3 if head == "paper" else 1) + 8 * B, 2.0 * n * B


def work(case):
    c, k = case, case["kind"]
    if k == "attn":
        lens = _lens(c)
        if c["branch"] == "local":
            counts = [_local_count(n, c["sink"], c["window"]) for n in lens]
        else:
            ranks = _flagged_ranks(c) or range(c["B"])
            counts = [min(lens[r], c["window"] or lens[r]) for r in ranks]
        return dict(bytes=_kv_bytes(c, counts) + _attn_io(c, len(counts)),
                    flops=4.0 * sum(counts) * c["L"] * c["Hq"] * c["D"])
    if k == "step":
        lens = _lens(c)
        counts = [_local_count(n, c["sink"], c["window"]) for n in lens]
        full = [lens[r] for r in _flagged_ranks(c)]
        gb, gf = _gate_work("paper", c["d"], c["dt"], c["B"])
        return dict(bytes=_kv_bytes(c, counts + full) + _attn_io(c, len(counts) + len(full)) + gb,
                    flops=4.0 * sum(counts + full) * c["L"] * c["Hq"] * c["D"] + gf)
    if k == "gate":
        b, f = _gate_work(c["head"], c["d"], c["dt"], c["B"])
        return dict(bytes=b, flops=f)
    if k == "mlp":
        B = c["listed"] or c["B"]
        n = 3.0 * c["d"] * c["F"]
        return dict(bytes=2 * n + 12.0 * B * c["d"] + 8.0 * B * c["F"] + 4 * c["d"], flops=2 * n * B)
    if k == "vocab":
        n = 1.0 * c["d"] * c["V"]
        return dict(bytes=2 * n + 4.0 * c["B"] * (c["d"] + c["V"]), flops=2 * n * c["B"])
    if k == "commit":
        row = 1.0 * c["L"] * c["B"] * c["Hkv"] * c["D"] * 4      # K and V, bf16
        return dict(bytes=3 * row, flops=0)
    # decoder
    s = _decoder_shape(c)
    gb, gf = _gate_work("paper", c["d"], c["dt"], c["B"])
    lens = _lens(c)
    counts = [_local_count(n, c["sink"], c["window"]) for n in lens]
    full = [lens[r] for r in _flagged_ranks(c)]
    head = 2.0 * s.vocab * s.d_model
    layers = float(s.weight_bytes()) - head
    passes = 2 if full else 1                                    # the retry streams the layers' weights again
    return dict(bytes=passes * layers + head + gb + _kv_bytes(c, counts + full) + 4.0 * c["B"] * s.vocab,
                flops=(layers * (c["B"] + len(full)) + head * c["B"])
                + 4.0 * sum(counts + full) * c["L"] * c["Hq"] * c["D"] + gf)


def tolerance(case):
    k = case["kind"]
    if k == "commit":
        return "exact"
    if k == "decoder":
        # fp32 sums in another order change a few bf16 roundings of q, k and v, and these travel
        # through the layers that follow
        return {"rel": 1e-3, "max": 2e-2}
    if k == "attn" and case["form"] == "qkv":
        # k_out and v_out are bf16: the fp32 norm and rotation may fall on the other side of a tie
        return {"rel": 1e-4, "max": 1e-2}
    if k == "gate":
        # a score is one value near a sum of terms of about 0.3
        return {"rel": 3e-5, "max": 3e-4}
    return {"rel": 1e-5, "max": 1e-4}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) * 1000003 + 17)
        self.cpu = torch.Generator()
        self.cpu.manual_seed(int(seed) * 1000003 + 17)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=torch.float32):
        t = torch.empty(*shape, dtype=dtype, device="cuda")
        flat = t.view(-1)
        step = 1 << 28
        for s in range(0, flat.numel(), step):
            flat[s:s + step].normal_(mean, std, generator=self.g)
        return t

    def bf16(self, *shape, std=1.0):
        return self.normal(*shape, std=std, dtype=torch.bfloat16)

    def perm(self, n):
        return torch.randperm(n, generator=self.cpu)


def _i32(v):
    return torch.as_tensor(v, dtype=torch.int32).cuda()


class _State:
    pass


def _deal(c, r, s):
    """Lengths dealt to the requests, the flagged requests, the block table."""
    lens, order = _lens(c), r.perm(c["B"]).tolist()
    s.lens = [lens[k] for k in order]
    flagged = set(_flagged_ranks(c))
    s.flagged = [b for b in range(c["B"]) if order[b] in flagged]
    s.max_len = c["hi"] + 1
    s.mb = -(-s.max_len // BLOCK)
    need = [-(-(n + 1) // BLOCK) for n in s.lens]
    s.nb = sum(need)
    ids = r.perm(s.nb)
    table = torch.zeros(c["B"], s.mb, dtype=torch.int32)
    at = 0
    for b, k in enumerate(need):
        table[b, :k] = ids[at:at + k]
        at += k
    s.table, s.seq = table.cuda(), _i32(s.lens)
    s.work = _i32(s.flagged + [0] * (c["B"] - len(s.flagged)))
    s.n_work = _i32([len(s.flagged)])


def _caches(c, r, s):
    s.k = r.bf16(c["L"], s.nb, c["Hkv"], c["D"] // 8, BLOCK, 8)
    s.v = r.bf16(c["L"], s.nb, c["Hkv"], c["D"], BLOCK)


def _shape(c, s):
    return P.Shape(c["L"], c["B"], c["Hq"], c["Hkv"], c["D"], s.mb, s.max_len, s.nb)


def _workspace(n):
    return torch.zeros(max(256, n), dtype=torch.uint8, device="cuda")


def _gate_inputs(c, r, s, head):
    """Packed parameters (weights and biases 0.02 N(0,1), gains 1 + 0.02 N(0,1)) and hidden states."""
    d, dt, B = c["d"], c["dt"], c["B"]
    s.params = r.normal(_gate_params(head, d, dt), std=0.02)
    for a, n in _gain_spans(head, d, dt):
        s.params[a:a + n] += 1.0
    s.h_prev, s.emb, s.h_local = r.normal(B, d), r.normal(B, d), r.normal(B, d)
    s.score = torch.zeros(B, device="cuda")
    s.flags = torch.zeros(B, dtype=torch.int32, device="cuda")
    s.gate = P.gate_desc(P.HEAD_PAPER if head == "paper" else P.HEAD_MLP, d, dt, s.params, EPS)
    s.ws_gate = _workspace(P.gate_workspace_size(s.gate, B))


def _gain_spans(head, d, dt):
    if head != "paper":
        return []
    tower, block = d + dt * d + dt, dt + 6 * dt * dt
    b0 = 3 * tower + 9 * dt * dt + dt
    return [(t * tower, d) for t in range(3)] + [(b0 + k * block, dt) for k in range(2)] + [(b0 + 2 * block, dt)]


def _prepare_attn(c, r, s):
    _deal(c, r, s)
    _caches(c, r, s)
    L, B, Hq, Hkv, D = c["L"], c["B"], c["Hq"], c["Hkv"], c["D"]
    s.out = torch.zeros(L, B, Hq, D, device="cuda")
    s.lse = torch.zeros(L, B, Hq, device="cuda")
    s.outputs = [s.out, s.lse]
    shape, scale = _shape(c, s), 1.0 / math.sqrt(D)
    local = c["branch"] == "local"
    ws = _workspace(P.attn_workspace_size(shape, c["sink"], c["window"]))
    wl = (s.work, s.n_work) if c["listed"] else (None, None)
    if c["form"] == "qkv":
        s.qkv = r.normal(B, (Hq + 2 * Hkv) * D)
        s.qg, s.kg = r.normal(D, std=0.02, mean=1.0), r.normal(D, std=0.02, mean=1.0)
        s.k_out = torch.zeros(B, Hkv, D, dtype=torch.bfloat16, device="cuda")
        s.v_out = torch.zeros_like(s.k_out)
        s.outputs += [s.k_out, s.v_out]
        inp = P.inputs(None, s.k, s.v, s.table, s.seq, scale)
        prep = P.qkv_prep(s.qkv, s.qg, s.kg, EPS, THETA, s.k_out, s.v_out)
        s.calls = [P.prepare_local_qkv(shape, inp, prep, c["sink"], c["window"], s.out, s.lse, ws) if local else
                   P.prepare_full_qkv(shape, inp, prep, c["window"], None, *wl, s.out, s.lse, ws)]
        return
    s.q = r.bf16(L, B, Hq, D)
    s.kc = s.vc = None
    if c["form"] == "cur":
        s.kc, s.vc = r.bf16(L, B, Hkv, D), r.bf16(L, B, Hkv, D)
    inp = P.inputs(s.q, s.k, s.v, s.table, s.seq, scale, s.kc, s.vc)
    s.calls = [P.prepare_local(shape, inp, c["sink"], c["window"], s.out, s.lse, ws) if local else
               P.prepare_full(shape, inp, c["window"], None, *wl, s.out, s.lse, ws)]


def _prepare_step(c, r, s):
    _deal(c, r, s)
    _caches(c, r, s)
    L, B, Hq, Hkv, D = c["L"], c["B"], c["Hq"], c["Hkv"], c["D"]
    shape = _shape(c, s)
    n = P.ring_elements(shape, c["sink"], c["window"])
    s.kr, s.vr = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    P.ring_fill(shape, s.k, s.v, s.table, s.seq, c["sink"], c["window"], s.kr, s.vr)
    s.q, s.kc, s.vc = r.bf16(L, B, Hq, D), r.bf16(L, B, Hkv, D), r.bf16(L, B, Hkv, D)
    s.out = torch.zeros(L, B, Hq, D, device="cuda")
    s.lse = torch.zeros(L, B, Hq, device="cuda")
    _gate_inputs(c, r, s, "paper")
    forced = torch.zeros(B, dtype=torch.int32)
    forced[s.flagged] = 1
    s.forced = forced.cuda()
    inp = P.inputs(s.q, s.k, s.v, s.table, s.seq, 1.0 / math.sqrt(D), s.kc, s.vc)
    s.calls = [P.prepare_local_ring(shape, inp, s.kr, s.vr, c["sink"], c["window"], s.out, s.lse,
                                    _workspace(P.attn_workspace_size(shape, c["sink"], c["window"]))),
               P.prepare_gate(s.gate, B, s.h_prev, s.emb, s.h_local, 0.0, s.forced, s.score, s.flags, s.work, s.n_work,
                              None, s.ws_gate),
               P.prepare_full(shape, inp, 0, None, s.work, s.n_work, s.out, s.lse,
                              _workspace(P.attn_workspace_size(shape, 0, 0)))]
    s.outputs = [s.out, s.lse, s.score, s.flags, s.work, s.n_work]


def _prepare_gate(c, r, s):
    _gate_inputs(c, r, s, c["head"])
    s.work = torch.zeros(c["B"], dtype=torch.int32, device="cuda")
    s.n_work = torch.zeros(1, dtype=torch.int32, device="cuda")
    s.calls = [P.prepare_gate(s.gate, c["B"], s.h_prev, s.emb, s.h_local, 0.05, None, s.score, s.flags, s.work, s.n_work,
                              None, s.ws_gate)]
    s.outputs = [s.score, s.flags, s.work, s.n_work]


def _prepare_mlp(c, r, s):
    d, F, B, k = c["d"], c["F"], c["B"], c["listed"]
    s.w_gu, s.w_down = r.bf16(2 * F, d, std=d ** -0.5), r.bf16(d, F, std=F ** -0.5)
    s.gain = r.normal(d, std=0.02, mean=1.0)
    s.h = r.normal(B, d)
    s.mlp = torch.zeros(B, F, device="cuda")
    s.y = torch.zeros(B, d, device="cuda")
    s.rows = sorted(r.perm(B).tolist()[:k]) if k else list(range(B))
    wl = (_i32(s.rows + [0] * (B - k)), _i32([k])) if k else (None, None)
    s.calls = [P.prepare_dense(P.dense_desc(d, F, P.DENSE_SWIGLU, s.w_gu, s.gain, EPS), B, s.h, None, s.mlp, *wl),
               P.prepare_dense(P.dense_desc(F, d, P.DENSE_PLAIN, s.w_down), B, s.mlp, s.h, s.y, *wl)]
    s.outputs = [s.mlp, s.y]


def _prepare_vocab(c, r, s):
    d, V, B = c["d"], c["V"], c["B"]
    s.w, s.x = r.bf16(V, d), r.normal(B, d)
    s.logits = torch.zeros(B, V, device="cuda")
    s.index = torch.zeros(B, dtype=torch.int32, device="cuda")
    s.calls = [P.prepare_dense(P.dense_desc(d, V, P.DENSE_PLAIN, s.w), B, s.x, None, s.logits),
               P.prepare_argmax(B, V, s.logits, s.index)]
    s.outputs = [s.logits, s.index]


def _prepare_commit(c, r, s):
    _deal(dict(c, listed=max(1, c["B"] // 8)), r, s)
    _caches(c, r, s)
    L, B, Hkv, D = c["L"], c["B"], c["Hkv"], c["D"]
    shape = P.Shape(L, B, Hkv, Hkv, D, s.mb, s.max_len, s.nb)
    n = P.ring_elements(shape, c["sink"], c["window"])
    s.kr, s.vr = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    P.ring_fill(shape, s.k, s.v, s.table, s.seq, c["sink"], c["window"], s.kr, s.vr)
    s.cand = [r.bf16(L, B, Hkv, D) for _ in range(4)]
    flags = torch.zeros(B, dtype=torch.int32)
    flags[s.flagged] = 1
    s.flags = flags.cuda()
    s.shape, s.sink, s.window = shape, c["sink"], c["window"]
    s.outputs = [s.k, s.v, s.kr, s.vr]


def _decoder_shape(c):
    return DecoderShape(c["L"], c["d"], c["Hq"], c["Hkv"], c["D"], c["F"], c["V"], EPS, THETA)


def _decoder_weights(c, r):
    L, d, Hq, Hkv, D, F, V = (c[k] for k in ("L", "d", "Hq", "Hkv", "D", "F", "V"))
    gain = lambda *shape: r.normal(*shape, std=0.02, mean=1.0)  # noqa: E731
    return dict(embed=r.bf16(V, d), attn_norm=gain(L, d), w_qkv=r.bf16(L, (Hq + 2 * Hkv) * D, d, std=d ** -0.5),
                q_norm=gain(L, D), k_norm=gain(L, D), w_o=r.bf16(L, d, Hq * D, std=(Hq * D) ** -0.5),
                mlp_norm=gain(L, d), w_gu=r.bf16(L, 2 * F, d, std=d ** -0.5), w_down=r.bf16(L, d, F, std=F ** -0.5),
                final_norm=gain(d))


def _prepare_decoder(c, r, s):
    _deal(c, r, s)
    _caches(c, r, s)
    B = c["B"]
    s.w = _decoder_weights(c, r)
    _gate_inputs(c, r, s, "paper")
    s.tokens = torch.randint(0, c["V"], (B,), generator=r.cpu, dtype=torch.int32).cuda()
    dec = Decoder(_decoder_shape(c), s.w, B, s.k, s.v, s.table, s.seq.clone(), s.mb, s.max_len, s.nb, c["sink"],
                  c["window"], gate=s.gate, tau=0.0, prescribed=True)
    dec.tokens.copy_(s.tokens)
    forced = torch.zeros(B, dtype=torch.int32)
    forced[s.flagged] = 1
    dec.forced.copy_(forced)
    s.dec = dec

    def step():
        local, retry, out = dec.oda_stages()
        for call in local + (retry if s.flagged else []) + out:
            call()

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
        side.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    s.outputs = [dec.logits, dec.h_prev, dec.k_loc, dec.v_loc, dec.score, dec.flags, dec.next_token, dec.seq_lens]
    if s.flagged:
        s.outputs += [dec.k_full, dec.v_full]



_PREPARE = dict(attn=_prepare_attn, step=_prepare_step, gate=_prepare_gate, mlp=_prepare_mlp, vocab=_prepare_vocab,
                commit=_prepare_commit, decoder=_prepare_decoder)


def prepare(case, seed):
    s = _State()
    s.kind = case["kind"]
    with torch.no_grad():
        _PREPARE[s.kind](case, _Rand(seed), s)
    return s


def run(s):
    if s.kind == "decoder":
        # the slots' state at the start of the step, then the step
        s.dec.seq_lens.copy_(s.seq)
        s.dec.h_prev.copy_(s.h_prev)
        s.graph.replay()
    elif s.kind == "commit":
        P.commit_kv_ring(s.shape, s.k, s.v, s.table, s.seq, *s.cand, flags=s.flags, advance=False, k_ring=s.kr,
                         v_ring=s.vr, n_sink=s.sink, window=s.window)
    else:
        for call in s.calls:
            call()
    return s.outputs


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _f64(t):
    return t.double()


def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * _f64(gain)


def _silu(x):
    return x * torch.sigmoid(x)


def _positions(c, branch, n):
    if branch == "local":
        start = max(min(c["sink"], n), n - c["window"])
        return list(range(min(c["sink"], n))) + list(range(start, n))
    w = c["window"] if c["kind"] == "attn" else 0
    return list(range(max(0, n - w) if w else 0, n))


def _attend(c, s, branch, layer, b, q, cur):
    """out [Hq][D] and lse [Hq] of one request; q, cur = (k, v) in 64 bits (cur None: all positions are cached)."""
    Hkv, D = c["Hkv"], c["D"]
    n = s.lens[b]
    pos = torch.tensor(_positions(c, branch, n), device="cuda")
    if cur is not None:
        pos = pos[pos < n - 1]
    lo, hi = (int(pos.min()), int(pos.max()) + 1) if len(pos) else (0, 0)
    blocks = s.table[b, :-(-hi // BLOCK)].long() if hi else s.table[b, :0].long()
    used = torch.unique(pos // BLOCK)
    at = torch.zeros(len(blocks), dtype=torch.long, device="cuda")
    at[used] = torch.arange(len(used), device="cuda")
    kb, vb = s.k[layer][blocks[used]], s.v[layer][blocks[used]]
    row = at[pos // BLOCK] * BLOCK + pos % BLOCK
    k = kb.permute(0, 3, 1, 2, 4).reshape(-1, Hkv, D)[row]
    v = vb.permute(0, 3, 1, 2).reshape(-1, Hkv, D)[row]
    k, v = _f64(k), _f64(v)
    if cur is not None:
        k, v = torch.cat([k, cur[0][None]]), torch.cat([v, cur[1][None]])
    qg = q.reshape(Hkv, -1, D)
    z = torch.matmul(qg, k.permute(1, 2, 0).contiguous()) / math.sqrt(D)
    lse = torch.logsumexp(z, -1)
    o = torch.matmul(torch.exp(z - lse[..., None]), v.permute(1, 0, 2).contiguous())
    return o.reshape(-1, D), lse.reshape(-1)


def _head(c, s, head, h_prev, emb, h_local):
    """Recall scores in 64 bits from the packed parameters."""
    d, dt = c["d"], c["dt"]
    p, at = s.params, [0]

    def take(*shape):
        n = math.prod(shape)
        v = _f64(p[at[0]:at[0] + n]).view(*shape)
        at[0] += n
        return v

    if head != "paper":
        w1, b1, w2, b2 = take(dt, d), take(dt), take(dt), take(1)
        z = h_local @ w1.T + b1
        return (0.5 * z * (1 + torch.erf(z / math.sqrt(2.0)))) @ w2 + b2
    abc = []
    for x in (h_prev, emb, h_local):
        g, w, b = take(d), take(dt, d), take(dt)
        abc.append(_silu(_rms(x, g) @ w.T + b))
    a, b, e = abc
    wf, bf = take(dt, 9 * dt), take(dt)
    u = torch.cat([a, b, e, a * b, (a - b).abs(), a * e, (a - e).abs(), b * e, (b - e).abs()], -1)
    z = 0.5 * (a + b + e + _silu(u @ wf.T + bf))
    for _ in range(2):
        g, wg, wu, wd = take(dt), take(2 * dt, dt), take(2 * dt, dt), take(dt, 2 * dt)
        n = _rms(z, g)
        z = z + (_silu(n @ wg.T) * (n @ wu.T)) @ wd.T
    g, wo, bo = take(dt), take(dt), take(1)
    return _rms(z, g) @ wo + bo


def _qkv64(c, qkv, qg, kg, n):
    """Query, key and value heads of one request's projection: norm and rotary embedding, before the bf16 rounding."""
    Hq, Hkv, D = c["Hq"], c["Hkv"], c["D"]
    x = qkv.view(-1, D)
    i = torch.arange(D // 2, device="cuda", dtype=torch.float64)
    ang = (n - 1) * THETA ** (-2 * i / D)
    co, si = torch.cos(ang), torch.sin(ang)

    def rope(x, gain):
        x = _rms(x, gain)
        a, b = x[:, :D // 2], x[:, D // 2:]
        return torch.cat([a * co - b * si, b * co + a * si], -1)

    return rope(x[:Hq], qg), rope(x[Hq:Hq + Hkv], kg), x[Hq + Hkv:]


def _bf(x):
    return _f64(x.float().bfloat16())


def _exact_attn(c, s):
    L, B, Hq, Hkv, D = c["L"], c["B"], c["Hq"], c["Hkv"], c["D"]
    out = torch.zeros(L, B, Hq, D, dtype=torch.float64, device="cuda")
    lse = torch.zeros(L, B, Hq, dtype=torch.float64, device="cuda")
    if c["form"] == "qkv":
        k_out = torch.zeros(B, Hkv, D, dtype=torch.float64, device="cuda")
        v_out = torch.zeros_like(k_out)
    for b in (s.flagged if c["listed"] else range(B)):
        for l in range(L):
            if c["form"] == "qkv":
                q, k_out[b], v_out[b] = _qkv64(c, _f64(s.qkv[b]), s.qg, s.kg, s.lens[b])
                q, cur = _bf(q), (_bf(k_out[b]), _bf(v_out[b]))
            else:
                q = _f64(s.q[l, b])
                cur = None if s.kc is None else (_f64(s.kc[l, b]), _f64(s.vc[l, b]))
            out[l, b], lse[l, b] = _attend(c, s, c["branch"], l, b, q, cur)
    return [out, lse] + ([k_out, v_out] if c["form"] == "qkv" else [])


def _exact_step(c, s):
    L, B, Hq, D = c["L"], c["B"], c["Hq"], c["D"]
    out = torch.zeros(L, B, Hq, D, dtype=torch.float64, device="cuda")
    lse = torch.zeros(L, B, Hq, dtype=torch.float64, device="cuda")
    for b in range(B):
        for l in range(L):
            out[l, b], lse[l, b] = _attend(c, s, "full" if b in s.flagged else "local", l, b, _f64(s.q[l, b]),
                                           (_f64(s.kc[l, b]), _f64(s.vc[l, b])))
    return [out, lse, _head(c, s, "paper", _f64(s.h_prev), _f64(s.emb), _f64(s.h_local)), None, None, None]


def _exact_gate(c, s):
    return [_head(c, s, c["head"], _f64(s.h_prev), _f64(s.emb), _f64(s.h_local)), None, None, None]


def _mlp64(h, gain, w_gu, w_down):
    n = _rms(h, gain)
    F = w_gu.shape[0] // 2
    m = _silu(n @ _f64(w_gu[:F]).T) * (n @ _f64(w_gu[F:]).T)
    return m, h + m @ _f64(w_down).T


def _exact_mlp(c, s):
    mlp = torch.zeros(c["B"], c["F"], dtype=torch.float64, device="cuda")
    y = torch.zeros(c["B"], c["d"], dtype=torch.float64, device="cuda")
    mlp[s.rows], y[s.rows] = _mlp64(_f64(s.h[s.rows]), s.gain, s.w_gu, s.w_down)
    return [mlp, y]


def _exact_vocab(c, s):
    return [_f64(s.x) @ _f64(s.w).T, None]


def _forward64(c, s, h, rows, branch):
    """Final hidden rows and the K/V candidates [L][rows] of one forward."""
    ks, vs = [], []
    w = s.w
    for l in range(c["L"]):
        qkv = _rms(h, w["attn_norm"][l]) @ _f64(w["w_qkv"][l]).T
        a, kl, vl = [], [], []
        for i, b in enumerate(rows):
            q, k, v = _qkv64(c, qkv[i], w["q_norm"][l], w["k_norm"][l], s.lens[b])
            kl.append(k)
            vl.append(v)
            a.append(_attend(c, s, branch, l, b, _bf(q), (_bf(k), _bf(v)))[0].reshape(-1))
        ks.append(torch.stack(kl))
        vs.append(torch.stack(vl))
        h = h + torch.stack(a) @ _f64(w["w_o"][l]).T
        h = _mlp64(h, w["mlp_norm"][l], w["w_gu"][l], w["w_down"][l])[1]
    return h, torch.stack(ks), torch.stack(vs)


def _exact_decoder(c, s):
    B = c["B"]
    emb = _f64(s.w["embed"][s.tokens.long()])
    h, kl, vl = _forward64(c, s, emb, range(B), "local")
    score = _head(c, s, "paper", _f64(s.h_prev), emb, _rms(h, s.w["final_norm"]))
    extra = []
    if s.flagged:
        hf, kf, vf = _forward64(c, s, emb[s.flagged], s.flagged, "full")
        h[s.flagged] = hf
        k_full, v_full = torch.zeros_like(kl), torch.zeros_like(vl)
        k_full[:, s.flagged], v_full[:, s.flagged] = kf, vf
        extra = [k_full, v_full]
    h = _rms(h, s.w["final_norm"])
    return [h @ _f64(s.w["embed"]).T, h, kl, vl, score, None, None, None] + extra


def exact(case, seed):
    fn = dict(attn=_exact_attn, step=_exact_step, gate=_exact_gate, mlp=_exact_mlp, vocab=_exact_vocab,
              decoder=_exact_decoder).get(case["kind"])
    if fn is None:
        return None      # the commit moves bytes
    with torch.no_grad():
        return fn(case, prepare(case, seed))

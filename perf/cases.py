"""The calls this library is measured on: its entry points over the sizes they are used at.

Five kinds of case, each one call (or, for "stream", one pass of the forward proxy) through the public entry points:

  materialize  fluxmoe_materialize / fluxmoe_materialize_two_streams: compressed experts -> staging slots
  ffn          fluxmoe_expert_ffn: the routed SwiGLU FFN over materialized slots
  shared       fluxmoe_shared_expert_ffn: the always-on expert on dense resident weights
  stream       harness.StreamingProxy: layers in waves, three streams, a share of the pool in pinned host memory
  encode       fluxmoe_encode_pool: offline compression (host buffers in, host blob out)

Layer shapes are those of paper_2604_02715_amd/inputs.py: hidden 4096 / ffn 14336 / 8 experts / top-2, hidden 2048 /
ffn 512 / 512 experts / top-10, hidden 5120 / ffn 1536 / 160 experts / top-8.  Weights, activations and routing follow the
same recipes as there, drawn here from the seed alone.
"""
import math

import numpy as np
import torch

from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs

DEVICE = "cuda:0"
COMPRESSED = 0.706          # compressed / dense bytes of the weight recipe, 4 KiB framing included


# ------------------------------------------------------------------------------------------ cases
def listed():
    return [
        # -- loading path
        # the smallest layer of the configurations: one call of a few microseconds, all launch and start-up
        dict(name="materialize_tiny", kind="materialize", experts=8, listed=8, hidden=256, ffn=512, two_streams=False),
        # one decode token at batch size one asks for its ten experts of 6 MB
        dict(name="materialize_token", kind="materialize", experts=32, listed=10, hidden=2048, ffn=512, two_streams=False),
        # a whole layer of few large experts (2.8 GB dense): the benchmark's default step
        dict(name="materialize_layer", kind="materialize", experts=8, listed=8, hidden=4096, ffn=14336, two_streams=False),
        # the 20-expert shard one GPU holds of a 160-expert layer, a stream for each tensor type (the paper's loading path)
        dict(name="materialize_shard", kind="materialize", experts=20, listed=20, hidden=5120, ffn=1536, two_streams=True),
        # -- FFN, decode
        # one token, top-10 of 512 small experts: the latency of a decode step at batch size one
        dict(name="ffn_token", kind="ffn", experts=512, hidden=2048, ffn=512, tokens=1, top_k=10, routing="zipf", mapped=512),
        # a decode batch on few large experts: every expert is touched, 64 rows each
        dict(name="ffn_decode", kind="ffn", experts=8, hidden=4096, ffn=14336, tokens=256, top_k=2, routing="softmax", mapped=8),
        # sizes that are multiples of nothing but 8 (an eighth of 2880 columns as a tensor-parallel slice), odd batch
        dict(name="ffn_ragged", kind="ffn", experts=64, hidden=2880, ffn=360, tokens=333, top_k=4, routing="uniform", mapped=64),
        # -- FFN, prefill
        # 1024 rows per expert on few large experts
        dict(name="ffn_prefill_large", kind="ffn", experts=8, hidden=4096, ffn=14336, tokens=4096, top_k=2, routing="softmax", mapped=8),
        # about 200 rows per expert on 160 experts with a short inner dimension
        dict(name="ffn_prefill_many", kind="ffn", experts=160, hidden=5120, ffn=1536, tokens=4096, top_k=8, routing="uniform", mapped=160),
        # the shared expert of that layer over a decode batch: a single expert, every token
        dict(name="shared_decode", kind="shared", hidden=5120, ffn=1536, tokens=512),
        # -- whole pass: three layers in waves through two slot halves, 2 % of the blocks from pinned host memory
        dict(name="stream_pass", kind="stream", layers=3, experts=128, hidden=2048, ffn=512, tokens=256, top_k=10,
             slots=64, routing="zipf", host_fraction=0.02),
        # -- offline compression of a few small experts (50 MB dense)
        dict(name="encode_experts", kind="encode", experts=8, hidden=2048, ffn=512),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _shape(rng):
    """(experts, hidden, ffn) around the three layer shapes: whole, an expert-parallel shard or a tensor-parallel slice, or ragged."""
    experts, hidden, ffn = rng.choice([(8, 4096, 14336), (512, 2048, 512), (160, 5120, 1536)])
    how = rng.choice(["whole", "shard", "slice", "ragged"])
    if how == "shard":
        experts = max(2, experts // rng.choice([2, 4, 8]))
    elif how == "slice":
        ffn = ffn // rng.choice([2, 4, 8])
    elif how == "ragged":
        hidden = _log_int(rng, 256, 5120, 8)
        ffn = _log_int(rng, 128, 2 * ffn if ffn < 4096 else ffn, 8)
    return max(1, min(experts, int(7.5e9) // (6 * hidden * ffn))), hidden, ffn


def draw(rng):
    kind = rng.choice(["materialize", "materialize", "ffn", "ffn", "ffn", "ffn", "shared", "stream", "encode"])
    if kind == "materialize":
        experts, hidden, ffn = _shape(rng)
        sigma = 6 * hidden * ffn
        experts = max(1, min(experts, int(1.0e9) // sigma))
        return dict(kind=kind, experts=experts, listed=_log_int(rng, 1, experts), hidden=hidden, ffn=ffn,
                    two_streams=rng.random() < 0.3)
    if kind == "ffn":
        experts, hidden, ffn = _shape(rng)
        top_k = min(experts, rng.choice([1, 2, 4, 8, 10]))
        # no more flops than the prefill case on large experts
        most = max(1, min(16384, int(2.8e12 / (6.0 * hidden * ffn * top_k))))
        mapped = experts if rng.random() < 0.75 else max(1, experts // 2)
        return dict(kind=kind, experts=experts, hidden=hidden, ffn=ffn, tokens=_log_int(rng, 1, most), top_k=top_k,
                    routing=rng.choice(["softmax", "zipf", "uniform"]), mapped=mapped)
    if kind == "shared":
        _, hidden, ffn = _shape(rng)
        return dict(kind=kind, hidden=hidden, ffn=ffn, tokens=_log_int(rng, 1, 8192))
    if kind == "stream":
        experts = rng.choice([24, 48, 96])
        return dict(kind=kind, layers=rng.choice([2, 3]), experts=experts, hidden=8 * rng.randrange(64, 257),
                    ffn=8 * rng.randrange(16, 65), tokens=_log_int(rng, 16, 512), top_k=rng.choice([2, 4, 8]),
                    slots=2 * rng.randrange(experts // 8, experts // 2 + 1), routing=rng.choice(["zipf", "uniform"]),
                    host_fraction=rng.choice([0.0, 0.01, 0.02]))
    return dict(kind=kind, experts=rng.randrange(1, 9), hidden=8 * rng.randrange(16, 257), ffn=8 * rng.randrange(8, 65))


# ------------------------------------------------------------------------------------------ inputs
def _generator(device, *key):
    g = torch.Generator(device=device)
    h = 1469598103934665603
    for k in key:
        for byte in str(k).encode() + b"/":
            h = ((h ^ byte) * 1099511628211) & 0x7FFFFFFFFFFFFFFF
    g.manual_seed(h)
    return g


def _weights(seed, layer, expert, which, rows, cols):
    """One stored matrix [rows][cols] in BF16 on the GPU: N(0, 0.02^2) with a scale of its own for each row and 0.1 % of
    the entries sixteen times as large, which gives the exponent statistics of trained weights."""
    g = _generator(DEVICE, "w", seed, layer, expert, which)
    w = torch.randn(rows, cols, generator=g, device=DEVICE).mul_(0.02)
    w.mul_(torch.exp(0.5 * torch.randn(rows, 1, generator=g, device=DEVICE)))
    big = torch.rand(rows, cols, generator=g, device=DEVICE) < 1e-3
    return w.mul_(1.0 + 15.0 * big).to(torch.bfloat16)


def _expert(seed, layer, expert, hidden, ffn):
    """(w13 [2][H][F], w2 [F][H])"""
    return (torch.stack([_weights(seed, layer, expert, 1, hidden, ffn), _weights(seed, layer, expert, 3, hidden, ffn)]),
            _weights(seed, layer, expert, 2, ffn, hidden))


def _layer_on_host(seed, layer, experts, hidden, ffn):
    w13 = torch.empty(experts, 2, hidden, ffn, dtype=torch.bfloat16, device=DEVICE)
    w2 = torch.empty(experts, ffn, hidden, dtype=torch.bfloat16, device=DEVICE)
    for e in range(experts):
        a, b = _expert(seed, layer, e, hidden, ffn)
        w13[e], w2[e] = a, b
    return w13.cpu(), w2.cpu()


def _activations(seed, layer, tokens, hidden):
    g = _generator(DEVICE, "x", seed, layer)
    return torch.randn(tokens, hidden, generator=g, device=DEVICE).to(torch.bfloat16)


def _numpy_rng(*key):
    return np.random.Generator(np.random.Philox(np.random.SeedSequence([b for k in key for b in str(k).encode() + b"/"])))


def _routing(seed, layer, tokens, top_k, experts, law):
    """(ids int32 [T][K], gates float32 [T][K]): the top-k of a softmax with renormalised gates, or k distinct experts drawn
    by popularity (zipf: rank^-1.1; uniform) with the gates of a softmax over k logits."""
    rng = _numpy_rng("r", seed, layer)
    if law == "softmax":
        logits = rng.standard_normal((tokens, experts))
        ids = np.argsort(-logits, axis=1, kind="stable")[:, :top_k]
        gl = np.take_along_axis(logits, ids, axis=1)
    else:
        logp = -1.1 * np.log(rng.permutation(experts) + 1.0) if law == "zipf" else np.zeros(experts)
        gumbel = -np.log(-np.log(rng.random((tokens, experts))))
        ids = np.argsort(-(logp + gumbel), axis=1, kind="stable")[:, :top_k]
        gl = rng.standard_normal((tokens, top_k))
    gates = np.exp(gl - gl.max(axis=1, keepdims=True))
    gates /= gates.sum(axis=1, keepdims=True)
    return np.ascontiguousarray(ids, dtype=np.int32), np.ascontiguousarray(gates, dtype=np.float32)


def _slots(seed, slots, experts):
    """(mapped experts ascending, their slots): which of a layer's experts are resident, and where"""
    rng = _numpy_rng("s", seed)
    return (np.sort(rng.permutation(experts)[:slots]).astype(np.int32), rng.permutation(slots).astype(np.int32))


def _config(case, **kw):
    args = dict(name="perf", n_experts=case["experts"], hidden=case["hidden"], ffn=case["ffn"], tokens=1, top_k=1,
                n_slots=case["experts"], routing="uniform", outliers=True)
    args.update(kw)
    return inputs.LayerConfig(**args)


class State:
    """What a program holds between calls; gives the context back when it goes."""

    def __init__(self, **kw):
        self.pool = None
        self.__dict__.update(kw)

    def __del__(self):
        if self.pool is not None:
            self.pool.close()


_streams = []


def _three_streams():
    # one set for the process, as a serving loop has: streams created later can share a hardware queue
    if not _streams:
        _streams.extend(torch.cuda.Stream() for _ in range(3))
    return tuple(_streams)


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state.call(state)


# ------------------------------------------------------------------------------------------ materialize
def _prepare_materialize(case, seed):
    E, n, H, F = case["experts"], case["listed"], case["hidden"], case["ffn"]
    pool = harness.ExpertPool(_config(case, n_slots=n), DEVICE)
    w13, w2 = _layer_on_host(seed, 0, E, H, F)
    pool.bind_layer(0, pool.encode_layer(0, w13, w2), check=False)
    pool.slots13.zero_()
    pool.slots2.zero_()
    pool.reset_page_table()
    ids, slots = _slots(seed, n, E)
    return State(call=_run_materialize, pool=pool, ids=ids, slots=slots, two=case["two_streams"])


def _run_materialize(s):
    p, cur = s.pool, torch.cuda.current_stream()
    if s.two:
        _, second, _ = _three_streams()
        B.fluxmoe_materialize_two_streams(p.ctx, 0, s.ids, p.page_table.data_ptr(), s.slots, cur.cuda_stream, second.cuda_stream)
    else:
        B.fluxmoe_materialize(p.ctx, 0, s.ids, p.page_table.data_ptr(), s.slots, cur.cuda_stream)
    return {"slots13": p.slots13, "slots2": p.slots2, "page_table": p.page_table}


# ------------------------------------------------------------------------------------------ FFN
def _prepare_ffn(case, seed):
    E, H, F, T, K, mapped = (case[k] for k in ("experts", "hidden", "ffn", "tokens", "top_k", "mapped"))
    pool = harness.ExpertPool(_config(case, tokens=T, top_k=K, n_slots=mapped), DEVICE)
    who, where = _slots(seed, mapped, E)
    for e, slot in zip(who, where):                     # the slots as fluxmoe_materialize leaves them
        w13, w2 = _expert(seed, 0, int(e), H, F)
        pool.slot13(int(slot)).copy_(w13.view(torch.int16).reshape(-1))
        pool.slot2(int(slot)).copy_(w2.view(torch.int16).reshape(-1))
    table = np.full(E, -1, dtype=np.int32)
    table[who] = where
    pool.page_table.copy_(torch.from_numpy(table)[None])
    ids, gates = _routing(seed, 0, T, K, E, case["routing"])
    return State(call=_run_ffn, pool=pool, x=_activations(seed, 0, T, H), ids=torch.from_numpy(ids).to(DEVICE),
                 gates=torch.from_numpy(gates).to(DEVICE), out=torch.zeros(T, H, device=DEVICE), T=T, K=K,
                 flags=0 if mapped == E else B.FFN_SKIP_UNMAPPED)


def _run_ffn(s):
    B.fluxmoe_expert_ffn(s.pool.ctx, 0, s.x.data_ptr(), s.T, s.ids.data_ptr(), s.gates.data_ptr(), s.K,
                         s.pool.page_table.data_ptr(), s.out.data_ptr(), s.flags, torch.cuda.current_stream().cuda_stream)
    return s.out


def _prepare_shared(case, seed):
    H, F, T = case["hidden"], case["ffn"], case["tokens"]
    pool = harness.ExpertPool(_config(dict(case, experts=2), tokens=T, n_slots=1, shared_expert=True), DEVICE)
    w13, w2 = _expert(seed, 0, "shared", H, F)
    return State(call=_run_shared, pool=pool, w13=w13, w2=w2, x=_activations(seed, 0, T, H), out=torch.zeros(T, H, device=DEVICE), T=T)


def _run_shared(s):
    B.fluxmoe_shared_expert_ffn(s.pool.ctx, s.w13.data_ptr(), s.w2.data_ptr(), s.x.data_ptr(), s.T, s.out.data_ptr(), 0,
                                torch.cuda.current_stream().cuda_stream)
    return s.out


def _swiglu_rows(x, w13, w2):
    """The FFN of one expert in 64 bits; the SwiGLU product is rounded to BF16 as the entry point documents."""
    g, u = x @ w13[0].double(), x @ w13[1].double()
    h = (g / (1.0 + torch.exp(-g)) * u).to(torch.bfloat16)
    return h.double() @ w2.double()


def _exact_routed(case, seed, layer, mapped):
    E, H, F, T, K = (case[k] for k in ("experts", "hidden", "ffn", "tokens", "top_k"))
    ids, gates = _routing(seed, layer, T, K, E, case["routing"])
    x = _activations(seed, layer, T, H).double()
    ids, gates = torch.from_numpy(ids).to(DEVICE), torch.from_numpy(gates).to(DEVICE).double()
    out = torch.zeros(T, H, dtype=torch.float64, device=DEVICE)
    for e in mapped:
        t, k = (ids == int(e)).nonzero(as_tuple=True)
        if t.numel():
            w13, w2 = _expert(seed, layer, int(e), H, F)
            out.index_add_(0, t, gates[t, k, None] * _swiglu_rows(x[t], w13, w2))
    return out


# ------------------------------------------------------------------------------------------ streaming pass
def _prepare_stream(case, seed):
    N, E, H, F, T, K = (case[k] for k in ("layers", "experts", "hidden", "ffn", "tokens", "top_k"))
    cfg = _config(case, tokens=T, top_k=K, n_slots=case["slots"], n_layers=N, host_fraction=case["host_fraction"])
    pool = harness.ExpertPool(cfg, DEVICE)
    staged = 0
    for layer in range(N):
        w13, w2 = _layer_on_host(seed, layer, E, H, F)
        _, n_host = pool.bind_layer(layer, pool.encode_layer(layer, w13, w2), case["host_fraction"], check=False)
        staged = max(staged, n_host)
    if staged:
        pool.bind_staging(2 * (staged + 1) * 4096)
    pool.reset_page_table()
    outs = [torch.zeros(T, H, device=DEVICE) for _ in range(N)]
    proxy = harness.StreamingProxy(pool, [_routing(seed, layer, T, K, E, case["routing"]) for layer in range(N)],
                                   [_activations(seed, layer, T, H) for layer in range(N)], outs, seed=seed,
                                   streams=_three_streams())
    return State(call=_run_stream, pool=pool, proxy=proxy, outs=outs)


def _run_stream(s):
    cur, p = torch.cuda.current_stream(), s.proxy
    for st in (p.load_stream, p.infer_stream, p.copy_stream):
        st.wait_stream(cur)
    p.run_pass()
    cur.wait_stream(p.infer_stream)
    return s.outs


# ------------------------------------------------------------------------------------------ encode
def _prepare_encode(case, seed):
    w13, w2 = _layer_on_host(seed, 0, case["experts"], case["hidden"], case["ffn"])
    ctx = B.fluxmoe_create(1, case["experts"], case["hidden"], case["ffn"], 1)
    blob = torch.zeros(int(B.fluxmoe_query_sizes(ctx).layer_blob_bound), dtype=torch.uint8)
    return Encoder(ctx=ctx, w13=w13, w2=w2, blob=blob)


class Encoder:
    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        B.fluxmoe_destroy(self.ctx)

    @staticmethod
    def call(s):
        used = B.fluxmoe_encode_pool(s.ctx, 0, s.w13.data_ptr(), s.w2.data_ptr(), s.blob.data_ptr(), s.blob.numel(), 16)
        # the buffer past the blob's `used` bytes is never written
        return {"blob": s.blob, "used": used, "lengths": [B.fluxmoe_code_lengths(s.ctx, 0, t) for t in (1, 2)]}


# ------------------------------------------------------------------------------------------ what a pass needs, and how exact it is
def _touched(case, mapped):
    ids, _ = _routing(0, 0, case["tokens"], case["top_k"], case["experts"], case["routing"])
    here = np.isin(ids, mapped)
    return len(np.unique(ids[here])), int(here.sum())


def work(case):
    kind, H, F = case["kind"], case["hidden"], case["ffn"]
    sigma = 6 * H * F                                    # dense bytes of one expert
    if kind == "materialize":
        return {"bytes": case["listed"] * sigma * (1 + COMPRESSED), "flops": 0}
    if kind == "encode":
        return {"bytes": case["experts"] * sigma * (1 + COMPRESSED), "flops": 0}
    io = 6 * case["tokens"] * H                          # BF16 tokens in, FP32 rows out
    if kind == "shared":
        return {"bytes": sigma + io, "flops": 6.0 * case["tokens"] * H * F}
    mapped = np.arange(case["experts"]) if kind == "stream" else _slots(0, case["mapped"], case["experts"])[0]
    touched, pairs = _touched(case, mapped)
    io += 8 * case["tokens"] * case["top_k"]
    if kind == "ffn":
        return {"bytes": touched * sigma + io, "flops": 6.0 * pairs * H * F}
    # a materialized expert is written to its slot and read from there
    return {"bytes": case["layers"] * (touched * sigma * (2 + COMPRESSED) + io), "flops": case["layers"] * 6.0 * pairs * H * F}


def tolerance(case):
    if case["kind"] in ("materialize", "encode"):
        return "exact"                                   # the codec is lossless, its container fixed
    # FP32 sums; h elements that lie at a BF16 tie round either way between two orders of summation: 8e-6 to 9.3e-5 from
    # the 64-bit result over these sizes
    return {"rel": 4e-4}


def exact(case, seed):
    kind = case["kind"]
    if kind == "ffn":
        return _exact_routed(case, seed, 0, _slots(seed, case["mapped"], case["experts"])[0])
    if kind == "shared":
        H, F, T = case["hidden"], case["ffn"], case["tokens"]
        return _swiglu_rows(_activations(seed, 0, T, H).double(), *_expert(seed, 0, "shared", H, F))
    if kind == "stream":
        return [_exact_routed(case, seed, layer, range(case["experts"])) for layer in range(case["layers"])]
    return None                                          # bytes: compared as they are

"""Performance cases of the VL-Cache hot path: what a serving program asks of this package, from one tiny prompt to
the largest batch one GPU takes.

A case is one of three kinds of pass, all through paper_2410_23317_amd.pipeline.VLCachePath:
  compress  a prompt batch has just been prefilled: score, sparsity, budgets, eviction, and the first decode steps
            over the compressed cache (one launch over all layers each).  route "sweeps" takes the statistics from the
            scoring sweeps, route "fused" from the attention of the window rows.
  decode    a batch is answered: eviction from given scores and budgets (which also resets the append counts), then
            `steps` generated tokens.  form "layers" replays a HIP graph that holds one step, one launch per layer (how
            a model issues it); form "all" is one ragged launch over all layers per token.
  eager     compress, then decode with one Python call per layer and token: the smallest problem, where call and
            launch latency is all there is.
Shapes are those of workloads.CONFIGS and of the benchmark's prompt grid; the inputs follow the recipe of workloads/
(unit-normal tensors, sink keys scaled by 4, a temperature per layer), drawn on the device.
"""
import math

import numpy as np
import torch

import paper_2410_23317_amd as V
from paper_2410_23317_amd.pipeline import VLCachePath

_BASE = dict(kind="compress", B=1, L=32, Hq=32, Hkv=8, d=128, m=2944, tau=32, dtype="bf16", alpha_num=1, alpha_den=10,
             steps=1, route="sweeps", form="all", fp8=False, ragged=False, recent=False)
P_FILTER = 0.01


def _case(name, **kw):
    c = dict(_BASE, name=name)
    c.update(kw)
    return c


def listed():
    return [
        # The tiny fp32 configuration: two layers, eight tokens, every call issued from Python.  Pure latency.
        _case("tiny-f32", kind="eager", L=2, Hq=4, Hkv=2, d=64, m=512, tau=32, dtype="f32", steps=8),
        # One single-image prompt on the 7B shape: the benchmark's headline compression.
        _case("compress-7b-2944"),
        # Four multi-image prompts on the 7B shape.
        _case("compress-7b-b4-10368", B=4, m=10368, tau=64),
        # The longest prompt of the benchmark's grid (128K tokens, window of the last 50).
        _case("compress-7b-131072", m=131072, tau=50),
        # The 34B-class shape (seven query heads per KV head), a batch of four: the largest, with its first 16 tokens.
        _case("serve-34b-b4-10368", B=4, L=60, Hq=56, m=10368, tau=64, steps=16),
        # Eight requests of different prompt and window lengths in one padded batch, with the recent window of a tenth
        # of each layer's budget; the padded length is odd.
        _case("compress-ragged-b8-4099", B=8, m=4099, tau=100, ragged=True, recent=True),
        # Scores from the attention of the window rows (the fused route), two requests of odd length.
        _case("fused-7b-b2-9973", B=2, m=9973, tau=64, route="fused"),
        # A small model with 64-wide heads.
        _case("compress-d64-b2-4096", B=2, L=24, Hq=16, Hkv=4, d=64, m=4096, tau=50),
        # A hundred tokens for one single-image prompt, one launch per layer from a captured step.
        _case("decode-layers-7b-2944", kind="decode", form="layers", steps=100),
        # The same for the batch of four multi-image prompts.
        _case("decode-layers-7b-b4-10368", kind="decode", form="layers", B=4, m=10368, tau=64, steps=32),
        # A hundred ragged launches over all layers, the benchmark's form, on the single-image prompt.
        _case("decode-all-7b-2944", kind="decode", steps=100),
        # The FP8 cache under a video prompt.
        _case("decode-all-fp8-7b-32768", kind="decode", m=32768, tau=64, fp8=True, steps=100),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads, KV heads, head dimension) of the drawn shapes: 1 to 8 query heads per KV head
_HEADS = [(32, 8, 128), (32, 8, 128), (32, 8, 128), (56, 8, 128), (16, 2, 128), (12, 4, 128), (8, 8, 128), (16, 4, 64)]


def draw(rng):
    kind = rng.choice(["compress", "compress", "compress", "decode", "decode", "decode", "eager"])
    alpha = rng.choice([(1, 10), (1, 10), (1, 20), (1, 5), (1, 100)])
    c = dict(_BASE, kind=kind, alpha_num=alpha[0], alpha_den=alpha[1])
    if kind == "eager":
        d, dtype = rng.choice([(64, "f32"), (128, "f32"), (128, "bf16"), (64, "bf16")])
        Hkv = rng.choice([1, 2, 4])
        c.update(B=rng.choice([1, 1, 2]), L=rng.randint(1, 4), Hkv=Hkv, Hq=Hkv * rng.choice([1, 2, 4]), d=d, dtype=dtype,
                 m=_log_uniform(rng, 128, 2048), tau=rng.randint(1, 64), steps=rng.randint(2, 8))
        return c
    c["Hq"], c["Hkv"], c["d"] = rng.choice(_HEADS)
    c["L"] = rng.randint(16, 60)
    # K rows of the whole batch: at most three quarters of the largest listed case's, and a tenth of that for 64-wide heads
    most = 15_000_000 if c["d"] == 128 else 1_500_000
    per = c["L"] * c["Hkv"]
    c["m"] = _log_uniform(rng, 512, min(131072, most // per))
    c["B"] = _log_uniform(rng, 1, max(1, min(32, most // (per * c["m"]))))
    c["tau"] = _log_uniform(rng, 8, 128)
    while c["tau"] > 16 and (c["Hq"] // c["Hkv"]) * c["tau"] * per * c["B"] * c["m"] > 7 * 64 * most:
        c["tau"] //= 2
    if kind == "compress":
        c["steps"] = rng.randint(1, 8)
        c["route"] = rng.choice(["sweeps", "sweeps", "fused"]) if c["d"] == 128 else "sweeps"
        c["ragged"] = c["B"] > 1 and rng.random() < 0.5
        c["recent"] = rng.random() < 0.3
    else:
        c["form"] = rng.choice(["layers", "all"])
        c["fp8"] = rng.random() < 0.3
        c["steps"] = rng.randint(16, 64)
    most_cost = max(_cost(x) for x in listed())
    while _cost(c) > most_cost:
        if c["steps"] > 8:
            c["steps"] //= 2
        else:
            c["m"] = c["m"] * 2 // 3
    return c


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


class State:
    pass


def prepare(case, seed):
    c = dict(_BASE, **case)
    B, L, Hq, Hkv, d, m, tau, T = (c[n] for n in ("B", "L", "Hq", "Hkv", "d", "m", "tau", "steps"))
    dev = torch.device("cuda")
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 2 + 1)
    host = np.random.default_rng([241023317, int(seed)])

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=dt)

    s = State()
    s.case = c
    s.k, s.v = normal(B, L, Hkv, m, d), normal(B, L, Hkv, m, d)
    n_sinks = 16
    pos = torch.randint(0, m, (B * L * Hkv, n_sinks), generator=gen, device=dev)
    flat = s.k.view(B * L * Hkv * m, d)
    at = torch.unique(torch.arange(B * L * Hkv, device=dev)[:, None] * m + pos)        # a position drawn twice is scaled once
    flat[at] = flat[at] * 4
    temperature = host.uniform(0.5, 2.0, L)
    s.sm = torch.from_numpy((1.0 / (temperature * math.sqrt(d))).astype(np.float32)).to(dev)
    s.dq, s.dk, s.dv = normal(T, L, B, Hq, d), normal(T, L, B, Hkv, d), normal(T, L, B, Hkv, d)
    s.out = torch.zeros((T, L, B, Hq, d), device=dev, dtype=dt)
    lens = None
    if c["ragged"]:
        mb = host.integers(max(1, m // 4), m + 1, B)
        tb = np.minimum(host.integers(max(1, tau // 4), tau + 1, B), mb)
        mb[0], tb[0] = m, tau
        lens = torch.from_numpy(np.stack([mb, tb], 1).astype(np.int32)).to(dev)
    shape = V.make_shape(B, L, Hq, Hkv, d, m, tau, c["dtype"], lens=lens)
    s.path = VLCachePath(shape, alpha=(c["alpha_num"], c["alpha_den"]), p=P_FILTER, T_max=T, want_idx=True, lens=lens,
                         recent_frac=(1, 10) if c["recent"] else None, kv_fp8=c["fp8"])
    s.path.cache.arena.zero_()
    if c["kind"] != "decode":
        s.q_win = normal(B, L, Hq, tau, d)
        s.win_out = torch.zeros_like(s.q_win)
        if c["ragged"]:                     # rows beyond a request's own window are left untouched
            s.path.row_max.zero_()
            s.path.row_sum.zero_()
        return s
    # decode: scores and budgets as a finished compression leaves them.  Budgets differ by layer as they do on the
    # workloads (a few layers at the lower clip, others at several times the mean).
    s.path.scores.copy_(torch.randn((B, L, Hkv, m), generator=gen, device=dev).exp_())
    w = host.uniform(0.0, 1.0, (B, L)) ** 2 + 1e-6
    total = (c["alpha_num"] * L * m) // c["alpha_den"]
    kk = np.clip(np.floor(w / w.sum(1, keepdims=True) * total), max(1, -(-m // 100)), m).astype(np.int32)
    s.budgets = torch.from_numpy(kk).to(dev)
    lay = s.path.cache.layout
    n_kv = B * lay.slots_per_request * 2 * Hkv * d * (1 if c["fp8"] else s.k.element_size())
    kv = s.path.cache.arena[lay.kv_off: lay.kv_off + n_kv]
    s.kv = kv if c["fp8"] else kv.view(dt)
    if c["form"] == "layers":
        # one decode step captured as a HIP graph: L launches on fixed buffers, the append count lives on the device
        s.step_q, s.step_k, s.step_v, s.step_out = s.dq[0], s.dk[0], s.dv[0], s.out[0]
        s.path.topk_compact(s.k, s.v, s.budgets)
        torch.cuda.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            for l in range(L):
                s.path.decode(l, l + 1, s.step_q[l], s.step_k[l], s.step_v[l], s.sm, s.step_out[l])
    return s


def run(s):
    c, path = s.case, s.path
    L, T = c["L"], c["steps"]
    if c["kind"] == "decode":
        path.topk_compact(s.k, s.v, s.budgets)
        if c["form"] == "layers":
            for _ in range(T):
                s.graph.replay()
            return {"out": s.step_out, "kv": s.kv, "idx": path.idx_out}
        path.decode_steps(0, L, T, s.dq, s.dk, s.dv, s.sm, s.out)
        return {"out": s.out, "kv": s.kv, "idx": path.idx_out}
    if c["route"] == "fused":
        path.window_attn(s.q_win, s.k, s.v, s.sm, s.win_out)
        path.score_from_stats(s.q_win, s.k, s.sm)
        path.sparsity()
        path.allocate()
        path.topk_compact(s.k, s.v)
    else:
        path.compress(s.q_win, s.k, s.v, s.sm)
    if c["kind"] == "eager":
        for t in range(T):
            for l in range(L):
                path.decode(l, l + 1, s.dq[t, l], s.dk[t, l], s.dv[t, l], s.sm, s.out[t, l])
    else:
        path.decode_steps(0, L, T, s.dq, s.dk, s.dv, s.sm, s.out)
    return {"scores": path.scores, "row_max": path.row_max, "row_sum": path.row_sum, "gamma": path.gamma, "beta": path.beta,
            "idx": path.idx_out, "window": s.win_out, "out": s.out}


def work(case):
    c = dict(_BASE, **case)
    B, L, Hq, Hkv, d, m, tau, T = (c[n] for n in ("B", "L", "Hq", "Hkv", "d", "m", "tau", "steps"))
    es = 4 if c["dtype"] == "f32" else 2
    rows = B * L * Hkv
    kept = B * L * m * c["alpha_num"] / c["alpha_den"] * Hkv                 # kept K rows of the batch (as many V rows)
    cached = d + 4 if c["fp8"] else d * es                                   # bytes of a cached row
    prompt = 0.62 if c["ragged"] else 1.0                                    # mean share of the padded prompt (and window) in use
    kept *= prompt
    evict = 4.0 * rows * m * prompt + 2 * kept * (d * es + cached) + 4 * kept          # scores, rows in and out, positions
    step = 2 * (kept + rows * (T + 1) / 2.0) * cached + B * L * (2 * Hq + 2 * Hkv) * d * es
    nbytes = evict + T * step
    flops = T * 4.0 * (kept + rows * (T + 1) / 2.0) * (Hq // Hkv) * d
    if c["kind"] != "decode":
        # the window's queries, K once (its kept rows are part of it), the scores out; the fused route also reads V and
        # writes the window's attention
        nbytes += (B * L * Hq * tau * d * es + rows * m * d * es) * prompt + 4.0 * rows * m - kept * d * es
        product = 2.0 * B * L * Hq * tau * m * d * prompt * prompt
        flops += product
        if c["route"] == "fused":
            nbytes += (rows * m * d * es + B * L * Hq * tau * d * es) * prompt - kept * d * es
            flops += product
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the path differs from itself by when its sums are taken in another order (the plain-ALU
    scoring and the generic window attention instead of the matrix cores; other unit sizes in decode): scores, row sums
    and the sparsity 1e-6, positions up to 1e-4 of the entries (a tie at the cut moves the entries between the two
    positions), bf16 outputs 1e-3.  fp32 storage: sums of a few hundred to a few thousand terms."""
    if case.get("dtype", "bf16") == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 5e-4}
    return {"rel": 4e-3, "max": 0.2, "differ": 5e-4}

"""The work that a user of this library has it do, as cases that can be timed.

Five kinds of work, all through the public entry points of paper_2504_09936_amd.binding:

  token     one decoded token through a stack of layers (keepkv_decode_step per layer) on compressed caches: a serving
            loop's inner step.  The pass first takes the token of the pass before off again (one small copy of the
            lengths, as a program does that rejects a drafted token), so that it can be repeated.
  generate  a compressed prefix is forked into the working caches (one copy), then a whole period is decoded, token by
            token through the layers, and every layer runs its compression event, compacting or in place.
  first     what follows a prefill: the window scores (keepkv_score_window), then the first event
            (keepkv_select, keepkv_match, keepkv_merge) from the whole context to the budget.
  prefill   the merge-first policy on a whole context: keepkv_prefill_match, keepkv_prefill_merge.
  full      decoding on the uncompressed cache (the time before the first event): keepkv_decode_attn, keepkv_score.

Shapes, ratios, periods, thresholds and key statistics are those of paper_2504_09936_amd/workloads.py and of the
benchmark; the inputs are drawn on the GPU from the seed.  With "graph" the launches are captured once, as the benchmark's
decode loop is, and a pass replays them; without, every call is made anew.
"""
import math

import torch

from paper_2504_09936_amd import binding as kk

ALPHA = 0.9               # EMA decay
N_SINK = 4                # tokens that selection always keeps
AR_RHO = 0.98             # 'ar1' keys: correlation of neighbours


def _case(name, kind, **kw):
    case = {"kind": kind, "dtype": "bf16", "batch": 1, "q_heads": 32, "kv_heads": 8, "head_dim": 128, "context": 8192,
            "budget": 820, "period": 64, "layers": 1, "window": 32, "causal": False, "keys": "outlier", "threshold": 0.8,
            "graph": False, "inplace": False, "ragged": False}
    case.update(kw)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest use: one layer of four f32 heads, one period of 32 tokens and its event, every call made anew
        _case("generate_tiny_f32", "generate", dtype="f32", q_heads=4, kv_heads=4, head_dim=64, context=512, budget=52,
              period=32),
        # interactive decoding of one sequence through 32 layers without a graph: launches and host time count
        _case("token_single_eager", "token", layers=32),
        # the headline shape: batch 8, 32 layers, captured
        _case("token_batch8", "token", batch=8, layers=32, graph=True),
        # a throughput server: batch 128, groups of eight query heads
        _case("token_batch128", "token", batch=128, q_heads=64, layers=4, keys="decay", graph=True),
        # the headline loop with its compacting events
        _case("generate_batch8", "generate", batch=8, layers=16, graph=True),
        # short periods, in-place events, slowly drifting keys
        _case("generate_inplace", "generate", batch=16, context=16384, period=16, layers=8, keys="ar1", graph=True,
              inplace=True),
        # after the prefill of a batch of 8 x 8192 tokens: few evicted keys find a partner
        _case("first_batch8", "first", batch=8),
        # after the prefill of one long document with many near-duplicates
        _case("first_long", "first", context=32768, budget=3277, period=128, keys="mixture", causal=True),
        # after the prefill of a large batch; strongly anisotropic keys: nearly every evicted key finds a partner
        _case("first_batch128", "first", batch=128, q_heads=64, window=8, keys="decay"),
        # a small model's narrow heads, sequences of different odd lengths
        _case("first_ragged", "first", batch=3, q_heads=16, head_dim=64, context=5003, budget=501, threshold=0.5,
              ragged=True),
        # merge-first prefill of the headline shape
        _case("prefill_batch8", "prefill", batch=8),
        # two sequences of 32768 tokens decoded on the uncompressed cache
        _case("full_long", "full", batch=2, context=32768, keys="mixture"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["token", "generate", "first", "prefill", "full"])
    keys = rng.choice(["outlier", "outlier", "mixture", "decay", "ar1"])
    f32 = rng.random() < 0.15
    head_dim = 64 if f32 or rng.random() < 0.25 else 128
    kv_heads = rng.choice([4, 8, 8, 8])
    q_heads = kv_heads * rng.choice([1, 2, 4, 4, 8])
    ratio = rng.uniform(0.05, 0.2)
    kw = {"dtype": "f32" if f32 else "bf16", "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim, "keys": keys,
          "ragged": rng.random() < 0.4, "threshold": rng.choice([0.8, 0.8, 0.5, -2.0])}
    if kind in ("token", "generate"):
        budget = _log_uniform(rng, 50, 3300)
        batch = _log_uniform(rng, 1, 4 if f32 else 128)
        while batch * budget > 128 * 900:
            batch = (batch + 1) // 2
        period = _log_uniform(rng, 16, 128)
        kw.update(batch=batch, budget=budget, context=int(budget / ratio), period=period, graph=rng.random() < 0.6,
                  layers=rng.randint(1, max(1, min(32, 100000 // (batch * budget)))), inplace=rng.random() < 0.5)
        if kind == "generate":
            kw["layers"] = max(1, min(kw["layers"], 768 // period))
    else:
        context = _log_uniform(rng, 512, 2048 if f32 else 32768)
        batch = _log_uniform(rng, 1, 4 if f32 else 64)
        most = {"first": 64 * 8192 * 8192, "prefill": 12 * 8192 * 8192, "full": 1 << 62}[kind]
        while batch * context * context > most or batch * context > 64 * 8192:
            batch -= 1 if batch < 8 else batch // 4
        kw.update(batch=max(1, batch), context=context, budget=max(52, min(4000, int(context * ratio))),
                  window=rng.choice([8, 16]) if q_heads // kv_heads == 8 else rng.choice([8, 16, 32]))
        kw["causal"] = kind == "first" and not kw["ragged"] and rng.random() < 0.5
    return _case(None, kind, **kw)


# ------------------------------------------------------------------------------------------------ inputs
def _keys_values(case, gen, lead, n):
    """n consecutive keys and values for every leading index (..., Hkv): float32 [*lead, n, D]."""
    D, shape = case["head_dim"], (*lead, n, case["head_dim"])
    k = torch.randn(shape, generator=gen, device="cuda")
    v = torch.randn(shape, generator=gen, device="cuda")
    if case["keys"] == "outlier":                       # a few channels of every head are six times as large
        ch = torch.rand((*lead, D), generator=gen, device="cuda").topk(4, dim=-1).indices
        gain = torch.ones((*lead, D), device="cuda").scatter_(-1, ch, 6.0)
        k *= gain.unsqueeze(-2)
    elif case["keys"] == "decay":                       # channel scales fall like 1 / channel, mean variance 1
        s = 1.0 / (1.0 + torch.arange(D, device="cuda", dtype=torch.float32))
        k *= s / s.square().mean().sqrt()
    elif case["keys"] == "mixture":                     # 64 clusters per head with a spread of 0.3 around unit centres
        mu = torch.nn.functional.normalize(torch.randn((*lead, 64, D), generator=gen, device="cuda"), dim=-1)
        which = torch.randint(64, (*lead, n), generator=gen, device="cuda")
        k *= 0.3
        k += torch.gather(mu, -2, which.unsqueeze(-1).expand(shape)) * math.sqrt(D)
    elif case["keys"] == "ar1":                         # neighbours correlate: y_i = rho y_(i-1) + c x_i, by doubling
        for x in (k, v):
            x[..., 1:, :] *= math.sqrt(1.0 - AR_RHO ** 2)
            s = 1
            while s < min(n, 1024):
                x[..., s:, :] += (AR_RHO ** s) * x[..., :-s, :].clone()
                s *= 2
    return k, v


def _queries(case, gen, lead):
    """Queries that look along one direction per head, with noise: [*lead, B, Hq, D]."""
    D, heads = case["head_dim"], (case["batch"], case["q_heads"], case["head_dim"])
    u = torch.nn.functional.normalize(torch.randn(heads, generator=gen, device="cuda"), dim=-1)
    xi = torch.randn((*lead, *heads), generator=gen, device="cuda")
    return (u + xi * (0.25 / math.sqrt(D))) * (3.0 * math.sqrt(D))


def _layout(case):
    return kk.Layout(case["batch"], case["q_heads"], case["kv_heads"], case["head_dim"],
                     kk.F32 if case["dtype"] == "f32" else kk.BF16, 1.0 / math.sqrt(case["head_dim"]))


def _views(cache, flat, layers):
    """The fields of `layers` caches like `cache`, carved from one buffer: {field: [layers, ...]}."""
    at, out = 0, {}
    for f in cache.FIELDS:
        t = getattr(cache, f)
        n = layers * t.numel() * t.element_size()
        out[f] = flat[at:at + n].view(t.dtype).view(layers, *t.shape)
        at += (n + 255) // 256 * 256
    return out, at


def _stack(case, lay, capacity):
    """Caches of all layers in one buffer, so that a program can fork or restore them with one copy."""
    one = kk.Cache(lay, capacity)
    layers = case["layers"]
    bytes_ = sum((layers * getattr(one, f).numel() * getattr(one, f).element_size() + 255) // 256 * 256 for f in one.FIELDS)
    flat = torch.zeros(bytes_, dtype=torch.uint8, device="cuda")
    fields, _ = _views(one, flat, layers)
    caches = []
    for layer in range(layers):
        c = kk.Cache(lay, 1)
        c.capacity = capacity
        for f in c.FIELDS:
            setattr(c, f, fields[f][layer])
        caches.append(c)
    return flat, fields, caches


def _fill_compressed(case, gen, fields, n_slots):
    """Caches as they are some time after a first event: merged slots with more votes, scores observed for a while."""
    shape = tuple(fields["votes"].shape)
    k, v = _keys_values(case, gen, shape[:-1], shape[-1])
    fields["k"].copy_(k)
    fields["v"].copy_(v)
    merged = torch.rand(shape, generator=gen, device="cuda") < 0.15
    fields["votes"].copy_(1 + merged * torch.randint(1, 20, shape, generator=gen, device="cuda"))
    t0 = 4 * case["window"]
    fields["t_obs"].fill_(t0)
    count = torch.randint(1, t0 + 1, shape, generator=gen, device="cuda")
    fields["born"].copy_(t0 - count)
    log_s = 1.5 * torch.randn(shape, generator=gen, device="cuda") + torch.log1p(-ALPHA ** count.float())
    fields["log_s"].copy_(log_s)
    if isinstance(n_slots, int):
        fields["len"].fill_(n_slots)
    else:
        fields["len"].copy_(n_slots)


class _State:
    pass


def _capture(fn):
    """`fn` once without a graph (it leaves the state as a pass would), then captured."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


def _prepare_token(case, gen, s):
    lay, B, H, P = s.lay, case["batch"], case["kv_heads"], case["period"]
    layers = case["layers"]
    s.flat, s.fields, s.caches = _stack(case, lay, case["budget"] + P)
    if case["ragged"]:
        n = case["budget"] + torch.randint(0, P, (layers, B, H), generator=gen, device="cuda")
        hint = case["budget"] + P - 1
    else:
        n = hint = case["budget"] + P // 2
    _fill_compressed(case, gen, s.fields, n)
    s.len0 = s.fields["len"].clone()
    q = _queries(case, gen, (layers,)).to(lay.torch_dtype)
    k, v = _keys_values(case, gen, (layers, B, H), 1)
    k, v = k[..., 0, :].to(lay.torch_dtype), v[..., 0, :].to(lay.torch_dtype)
    s.out = torch.zeros_like(q)
    s.ws = kk.new_workspace(lay, case["budget"] + P, case["budget"])
    for c in s.caches:
        c.len_hint = hint
    s.args = [(s.caches[i], q[i], k[i], v[i], s.out[i]) for i in range(layers)]

    def layers_once():
        for cache, q_t, k_t, v_t, out in s.args:
            kk.decode_step(lay, cache, q_t, k_t, v_t, out, None, ALPHA, None, s.ws)

    s.launch = _capture(layers_once).replay if case["graph"] else layers_once


def _run_token(s):
    s.fields["len"].copy_(s.len0)
    s.launch()
    return {"out": s.out, **s.fields}


def _prepare_generate(case, gen, s):
    lay, B, H, P, budget, layers = s.lay, case["batch"], case["kv_heads"], case["period"], case["budget"], case["layers"]
    cap = budget + P
    s.flat, s.fields, s.caches = _stack(case, lay, cap)
    _fill_compressed(case, gen, s.fields, budget)
    s.saved = s.flat.clone()
    n_recent = (4 * (budget - N_SINK)) // 5
    q = _queries(case, gen, (layers, P)).to(lay.torch_dtype)
    k, v = _keys_values(case, gen, (layers, B, H), P)
    k, v = (x.permute(0, 3, 1, 2, 4).to(lay.torch_dtype).contiguous() for x in (k, v))
    s.out = torch.zeros_like(q)
    s.ws = kk.new_workspace(lay, cap, budget)
    s.keep = torch.zeros(layers, B, H, budget, dtype=torch.int32, device="cuda")
    s.evict = torch.zeros(layers, B, H, P, dtype=torch.int32, device="cuda")
    s.match = torch.zeros_like(s.evict)
    s.n_ev = torch.zeros(layers, B, H, dtype=torch.int32, device="cuda")
    s.dropped = torch.zeros(layers, B, H, dtype=torch.int64, device="cuda")
    if case["inplace"]:
        s.order0 = torch.arange(budget, dtype=torch.int32, device="cuda").repeat(layers, B, H, 1).contiguous()
        s.order = s.order0.clone()
        s.result = {"order": s.order, **s.fields}
    else:
        s.dst_flat, dst_fields, s.dst = _stack(case, lay, cap)
        s.result = dst_fields
    s.steps = [[(s.caches[i], q[i, t], k[i, t], v[i, t], s.out[i, t]) for i in range(layers)] for t in range(P)]
    lists = [(s.keep[i], s.evict[i], s.n_ev[i], s.match[i], s.dropped[i]) for i in range(layers)]

    def event(i):
        keep, evict, n_ev, match, dropped = lists[i]
        c = s.caches[i]
        if case["inplace"]:
            kk.select_aged(lay, c, s.order[i], budget, N_SINK, n_recent, ALPHA, keep, evict, n_ev, s.ws)
            kk.match(lay, c, budget, keep, evict, n_ev, case["threshold"], match, None, s.ws)
            kk.merge_inplace(lay, c, s.order[i], budget, keep, evict, n_ev, match, ALPHA, dropped)
        else:
            kk.select(lay, c, budget, N_SINK, n_recent, ALPHA, keep, evict, n_ev, s.ws)
            kk.match(lay, c, budget, keep, evict, n_ev, case["threshold"], match, None, s.ws)
            kk.merge(lay, c, s.dst[i], budget, keep, evict, n_ev, match, ALPHA, dropped, s.ws)

    def period():
        for t, step in enumerate(s.steps):
            for i, (cache, q_t, k_t, v_t, out) in enumerate(step):
                cache.len_hint = budget + t
                kk.decode_step(lay, cache, q_t, k_t, v_t, out, None, ALPHA, None, s.ws)
                if t == P - 1:
                    event(i)

    s.launch = _capture(period).replay if case["graph"] else period
    s.dropped.zero_()


def _run_generate(s):
    s.flat.copy_(s.saved)
    if s.case["inplace"]:
        s.order.copy_(s.order0)
    s.launch()
    return {"out": s.out, "keep": s.keep, "evict": s.evict, "match": s.match, "n_evict": s.n_ev, "dropped": s.dropped,
            **s.result}


def _prefilled(case, gen, lay):
    B, H, N = case["batch"], case["kv_heads"], case["context"]
    cache = kk.Cache(lay, N)
    for b in range(0, B, 16):                            # (in parts: the f32 draws are twice the size)
        k, v = _keys_values(case, gen, (min(16, B - b), H), N)
        cache.k[b:b + 16].copy_(k)
        cache.v[b:b + 16].copy_(v)
    cache.votes.fill_(1)
    cache.len.fill_(N)
    if case["ragged"]:                                   # sequences of different lengths
        n = torch.randint(max(1, N // 2), N + 1, (B, 1), generator=gen, device="cuda")
        n[0] = N
        cache.len.copy_(n.expand(B, H))
    return cache


def _prepare_first(case, gen, s):
    lay, B, H, N, budget = s.lay, case["batch"], case["kv_heads"], case["context"], case["budget"]
    s.cache = _prefilled(case, gen, lay)
    s.q_win = _queries(case, gen, (case["window"],)).permute(1, 2, 0, 3).to(lay.torch_dtype).contiguous()
    s.n_recent = (4 * (budget - N_SINK)) // 5
    s.dst = kk.Cache(lay, budget + case["period"])
    s.keep = torch.zeros(B, H, budget, dtype=torch.int32, device="cuda")
    s.evict = torch.zeros(B, H, N - budget, dtype=torch.int32, device="cuda")
    s.match = torch.zeros_like(s.evict)
    s.n_ev = torch.zeros(B, H, dtype=torch.int32, device="cuda")
    s.dropped = torch.zeros(B, H, dtype=torch.int64, device="cuda")
    s.ws = kk.new_workspace(lay, N, budget)


def _run_first(s):
    case, lay, budget, W = s.case, s.lay, s.case["budget"], s.case["window"]
    per_call = min(W, 128 * case["kv_heads"] // case["q_heads"])
    first_pos = case["context"] - W if case["causal"] else -1
    for j in range(0, W, per_call):
        q = s.q_win if per_call == W else s.q_win[:, :, j:j + per_call].contiguous()
        kk.score_window(lay, s.cache, q, per_call, ALPHA, first_pos + j if case["causal"] else -1)
    kk.select(lay, s.cache, budget, N_SINK, s.n_recent, ALPHA, s.keep, s.evict, s.n_ev, s.ws)
    kk.match(lay, s.cache, budget, s.keep, s.evict, s.n_ev, case["threshold"], s.match, None, s.ws)
    kk.merge(lay, s.cache, s.dst, budget, s.keep, s.evict, s.n_ev, s.match, ALPHA, s.dropped, s.ws)
    return {"scores": s.cache.log_s, "keep": s.keep, "evict": s.evict, "match": s.match, "n_evict": s.n_ev,
            "dropped": s.dropped, **{f: getattr(s.dst, f) for f in s.dst.FIELDS}}


def _prepare_prefill(case, gen, s):
    lay, B, H, N = s.lay, case["batch"], case["kv_heads"], case["context"]
    s.cache = _prefilled(case, gen, lay)
    s.cache.log_s.copy_(1.5 * torch.randn((B, H, N), generator=gen, device="cuda"))
    s.cache.t_obs.fill_(case["window"])
    s.dst = kk.Cache(lay, N)
    s.near = torch.full((B, H, N), -1, dtype=torch.int32, device="cuda")
    s.ws = kk.new_workspace(lay, N, case["budget"])


def _run_prefill(s):
    kk.prefill_match(s.lay, s.cache, s.case["threshold"], s.near, None, s.ws)
    kk.prefill_merge(s.lay, s.cache, s.dst, s.near, ALPHA, s.ws)
    return {"near": s.near, **{f: getattr(s.dst, f) for f in s.dst.FIELDS}}


def _prepare_full(case, gen, s):
    lay, B, H, N = s.lay, case["batch"], case["kv_heads"], case["context"]
    s.cache = _prefilled(case, gen, lay)
    s.cache.log_s.copy_(1.5 * torch.randn((B, H, N), generator=gen, device="cuda"))
    s.cache.t_obs.fill_(case["window"])
    s.cache.len_hint = N
    s.q = _queries(case, gen, ()).to(lay.torch_dtype)
    s.out = torch.zeros_like(s.q)
    s.lse = torch.zeros(B, case["q_heads"], device="cuda")
    s.logits = torch.zeros(B, H, N, device="cuda")
    s.ws = kk.new_workspace(lay, N, case["budget"])


def _run_full(s):
    kk.decode_attn(s.lay, s.cache, s.q, s.out, s.logits, s.lse, s.ws)
    kk.score(s.lay, s.cache, s.logits, ALPHA)
    return {"out": s.out, "logits": s.logits, "lse": s.lse, "log_s": s.cache.log_s}


_PREPARE = {"token": _prepare_token, "generate": _prepare_generate, "first": _prepare_first, "prefill": _prepare_prefill,
            "full": _prepare_full}
_RUN = {"token": _run_token, "generate": _run_generate, "first": _run_first, "prefill": _run_prefill, "full": _run_full}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = _State()
    s.case, s.lay = case, _layout(case)
    _PREPARE[case["kind"]](case, gen, s)
    return s


def run(state):
    return _RUN[state.case["kind"]](state)


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _step_work(case, n_slots):
    """One decode step of one layer with n_slots attended slots per head."""
    e = 4 if case["dtype"] == "f32" else 2
    units, D = case["batch"] * case["kv_heads"], case["head_dim"]
    row = 2 * D * e
    heads = case["batch"] * case["q_heads"]
    return (units * (n_slots * (row + 12) + 2 * row) + 2 * heads * D * e, 4.0 * heads * n_slots * D)


def _event_work(case, n, V_read):
    """An event from n to budget slots per head; V_read: value rows that have to be read."""
    e = 4 if case["dtype"] == "f32" else 2
    units, D, budget = case["batch"] * case["kv_heads"], case["head_dim"], case["budget"]
    moved = n * D * e + V_read * D * e + n * 16 + n * 8 + budget * (2 * D * e + 12)
    return units * moved, 2.0 * units * (n - budget) * budget * D


def _mean_len(case):
    return case["context"] * 0.75 if case["ragged"] else case["context"]


def work(case):
    units, D, W = case["batch"] * case["kv_heads"], case["head_dim"], case["window"]
    e = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "token":
        b, f = _step_work(case, case["budget"] + case["period"] // 2)
        return {"bytes": case["layers"] * b, "flops": case["layers"] * f}
    if case["kind"] == "generate":
        budget, P = case["budget"], case["period"]
        b, f = _step_work(case, budget + P // 2)
        eb, ef = _event_work(case, budget + P, P if case["inplace"] else budget + P)
        fork = 2 * units * (budget + P) * (2 * D * e + 12)
        return {"bytes": case["layers"] * (P * b + eb + fork), "flops": case["layers"] * (P * f + ef)}
    n = _mean_len(case)
    if case["kind"] == "first":
        many = case["keys"] in ("decay", "mixture") or case["threshold"] < 0      # most evicted keys find a partner
        b, f = _event_work(case, n, n if many else case["budget"])
        return {"bytes": b + 8 * units * n, "flops": f + 2.0 * case["batch"] * case["q_heads"] * W * n * D}
    if case["kind"] == "prefill":
        return {"bytes": units * n * 2 * (2 * D * e + 12), "flops": 1.0 * units * n * n * D}
    b, f = _step_work(case, n)
    return {"bytes": b + 4 * units * n, "flops": f}


def tolerance(case):
    # Measured with the slots of every decode call split differently over the workgroups (another order of the softmax
    # and value sums): bf16 outputs differ by 2e-5 to 1.1e-4 (2-norm; single values by one bf16 step, 2^-7), f32 outputs
    # by 5e-8 to 8e-8; scores are sums of at most 128 exact products in f32, their logarithms move by about 1e-6.
    # Whole numbers agree unless such a difference decides between two nearly equal scores, which moves one list entry.
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4, "differ": 1e-3}
    return {"rel": 4.5e-4, "max": 0.035, "differ": 1e-3}

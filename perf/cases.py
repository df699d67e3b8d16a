"""The decode-step workloads whose speed counts, for timing and comparing builds of this repository.

One pass of a case is one generated token of a batch of audio chunks: the retained set of every sequence under its
eviction policy and the attention over it in every decoder layer, through the entry points of
`paper_2606_01483_amd.murmur`.  A decoder computes its layers one after the other, so most cases make one attention
call per layer, captured into a HIP graph once, as a serving program does (`graph`); the others make one call for
all layers of the token (`per_call` equal to `layers`) and issue it eagerly.

    api       step    murmur_decode_step (retained set inside the attention launch)
              ring    murmur_decode_step_ring (output ring storage, appends the current token)
              ranges  murmur_evict_compact once per token, then murmur_decode_attn with the range table
              index   the same with the index list
              paged   murmur_paged_step, murmur_evict_compact_paged, then murmur_decode_attn over the block pool

Caches, queries and current-token rows are drawn on the GPU from the seed; lengths come from the case alone.  Rows
that hold no token are bf16 NaN, so a stray read shows in the outputs.
"""
import math

import numpy as np
import torch

from paper_2606_01483_amd import murmur as M

D = 128           # head_dim
OFF = -1          # window value that keeps a whole region
NAN_BITS = 0x7FC0
PLANT_SHARE, PLANT_LIFT, PLANT_RHO = 0.05, 3.0, 0.8  # sparse speech attention, as the eviction workloads draw it

DEFAULTS = dict(api="step", layers=28, per_call=1, graph=True, batch=12, prompt=32, prompt_mid=0, speech_lo=2250,
                speech_hi=2250, out_lo=600, out_hi=1200, w_s=OFF, quarter=False, delay=0, sink_s=0, w_o=OFF, sink_o=0,
                dense_layers=0, hq=28, hkv=4, out_f32=False, lists=False, planted=False, block=0)


def _case(**kw):
    return dict(DEFAULTS, **kw)


def listed():
    evict = dict(w_s=562, delay=512, w_o=256, planted=True)
    return [
        # The smallest call: one minute of audio, one sequence, one layer, issued eagerly.  Latency and launch cost.
        _case(name="minute_one_call", layers=1, graph=False, batch=1, speech_lo=450, speech_hi=450, out_lo=72,
              out_hi=72, w_s=128, delay=72, w_o=32, lists=True, out_f32=True),
        # The same minute through a whole 28-layer decoder, one captured call per layer: interactive transcription.
        _case(name="minute_28_layers", batch=1, speech_lo=450, speech_hi=450, out_lo=72, out_hi=72, w_s=128, delay=72,
              w_o=32, out_f32=True),
        # The headline workload: 12 chunks of 300 s with eviction, a call per layer.
        _case(name="chunks12_evict", lists=True, **evict),
        # The same batch without eviction: the dense decode baseline, chunks of different output lengths.
        _case(name="chunks12_dense"),
        # An hour in a single pass, dense: one long sequence.
        _case(name="hour_dense", batch=1, speech_lo=27000, speech_hi=27000, out_lo=8064, out_hi=8064),
        # The hour with eviction: a few short windows of one sequence.
        _case(name="hour_evict", batch=1, speech_lo=27000, speech_hi=27000, out_lo=8064, out_hi=8064, w_s=2048,
              delay=512, w_o=512),
        # All 28 layers of the 12-chunk batch in one eager call, ragged chunks, speech window of a quarter.
        _case(name="stack28_evict", per_call=28, graph=False, speech_lo=1800, speech_hi=2250, out_lo=300, out_hi=1200,
              quarter=True, delay=512, w_o=256, planted=True, lists=True),
        # The same stack with its first four layers dense: policies per layer, groups of unequal length.
        _case(name="stack28_per_layer", per_call=28, graph=False, speech_lo=1800, speech_hi=2250, out_lo=300,
              out_hi=1200, quarter=True, delay=512, w_o=256, planted=True, dense_layers=4, out_f32=True),
        # The headline batch on ring storage: eviction frees memory, the step appends the current token.
        _case(name="chunks12_ring", api="ring", **evict),
        # The headline batch on a paged pool of 16-row blocks managed on the device.
        _case(name="chunks12_paged", api="paged", block=16, **evict),
        # A batch of 16 chunks at every stage of their decode, both windows of the ablations, range tables made once
        # per token and read by every layer.
        _case(name="chunks16_ranges", api="ranges", batch=16, out_lo=1, out_hi=2700, w_s=1024, delay=512, w_o=1024,
              sink_o=4),
        # Continuous batching: 64 chunks at every stage of their decode, no eviction.
        _case(name="serve64_dense", batch=64, out_lo=1, out_hi=2700),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any entry point, 1 to 64 sequences of a minute to an hour, 1 to 28 layers, any policy."""
    most = max(work(c)["bytes"] for c in listed())
    while True:
        api = rng.choice(["step", "step", "step", "ring", "paged", "ranges", "index"])
        hq, hkv = rng.choice([(28, 4), (28, 4), (28, 4), (28, 4), (16, 4), (16, 1), (8, 2), (4, 4)])
        batch = _log_int(rng, 1, 64)
        layers = _log_int(rng, 1, 28)
        per_call = rng.choice([1, 1, layers])
        speech_hi = _log_int(rng, 300, 27000)
        speech_lo = rng.choice([speech_hi, rng.randint(speech_hi // 3, speech_hi)])
        out_hi = _log_int(rng, 16, 8000)
        out_lo = rng.choice([out_hi, rng.randint(1, out_hi)])
        c = _case(api=api, hq=hq, hkv=hkv, batch=batch, layers=layers, per_call=per_call, graph=per_call < layers,
                  speech_lo=speech_lo, speech_hi=speech_hi, out_lo=out_lo, out_hi=out_hi, prompt=rng.randint(4, 64),
                  prompt_mid=rng.choice([0, 0, rng.randint(1, 40)]), out_f32=rng.random() < 0.5,
                  planted=rng.random() < 0.5, lists=api == "step" and rng.random() < 0.5)
        if rng.random() < 0.6:  # speech eviction
            c.update(w_s=_log_int(rng, 64, max(65, speech_hi)), delay=rng.choice([0, 256, 512]),
                     sink_s=rng.choice([0, 0, rng.randint(1, 64)]), quarter=rng.random() < 0.3)
        if rng.random() < 0.6 or api == "ring":  # output eviction
            c.update(w_o=_log_int(rng, 32, max(33, out_hi)), sink_o=rng.choice([0, 4, 8]))
        if api == "step" and per_call == layers and layers > 1 and rng.random() < 0.3:
            c.update(dense_layers=rng.randint(1, layers - 1))
        if api == "paged":
            c.update(block=rng.choice([8, 16, 64]))
        seg, _ = _layout(c)
        cache = layers * batch * int(seg.sum(axis=1).max()) * hkv * D * 4
        if work(c)["bytes"] <= 0.6 * most and cache <= 18e9:
            return c


# ---- lengths, policies and retained sets (plain numpy; one [B, 4] layout and one [B, 5] policy per layer) ----------

def _layout(c):
    rng = np.random.default_rng([c["batch"], c["speech_hi"], c["out_hi"], c["layers"]])
    b = c["batch"]
    speech = rng.integers(c["speech_lo"], c["speech_hi"], size=b, endpoint=True)
    out = rng.integers(c["out_lo"], c["out_hi"], size=b, endpoint=True)
    seg = np.stack([np.full(b, c["prompt"]), speech, np.full(b, c["prompt_mid"]), out], axis=1).astype(np.int32)
    w_s = np.maximum(speech // 4, 1) if c["quarter"] else np.full(b, c["w_s"])
    pol = np.stack([w_s, np.full(b, c["delay"]), np.full(b, c["sink_s"]), np.full(b, c["w_o"]),
                    np.full(b, c["sink_o"])], axis=1).astype(np.int32)
    dense = np.tile(np.array([OFF, 0, 0, OFF, 0], dtype=np.int32), (b, 1))
    return seg, [dense if layer < c["dense_layers"] else pol for layer in range(c["layers"])]


def _kept(seg, pol):
    """Retained positions of one sequence at its step out_len, ascending."""
    p0, ls, p1, j = (int(x) for x in seg)
    w_s, delay, sink_s, w_o, sink_o = (int(x) for x in pol)
    speech = np.ones(ls, dtype=bool)
    if w_s != OFF:
        lo = min(max(0, j - max(delay, 1) + 1), max(ls - w_s, 0))
        t = np.arange(ls)
        speech = (t < sink_s) | ((t >= lo) & (t < lo + w_s))
    out = np.ones(j, dtype=bool)
    if w_o != OFF:
        t = np.arange(j)
        out = (t < sink_o) | (t >= j - w_o)
    return np.flatnonzero(np.concatenate([np.ones(p0, bool), speech, np.ones(p1, bool), out]))


def _kept_counts(c):
    seg, pols = _layout(c)
    per = {}
    counts = []
    for pol in pols:
        if id(pol) not in per:
            per[id(pol)] = [len(_kept(seg[b], pol[b])) for b in range(c["batch"])]
        counts.append(per[id(pol)])
    return np.array(counts)  # [layers, batch]


def work(c):
    kept = _kept_counts(c)
    rows, hq, hkv, b = int(kept.sum()), c["hq"], c["hkv"], c["batch"]
    heads = c["layers"] * b * hq
    io = heads * (2 * D + (4 if c["out_f32"] else 2) * D + 4) + b * 36
    if c["lists"] or c["api"] in ("index", "paged"):
        io += b * int(kept.max()) * 4
    if c["api"] in ("ring", "paged"):
        io += 2 * c["layers"] * b * hkv * 2 * D * 2  # the current token's rows, read and appended
    return {"bytes": rows * hkv * 2 * D * 2 + io, "flops": rows * hq * D * 4}


def tolerance(c):
    # fp32 outputs: fp32 accumulation, weights carried to 16 mantissa bits.  bf16 outputs: half a bf16 step.
    return {"rel": 1e-5, "max": 2e-4} if c["out_f32"] else {"rel": 6e-3, "max": 2e-2}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed, *extra):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([seed, *extra]).generate_state(1, np.uint64)[0] >> 1))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _queries(c, seed):
    """bf16 [layers, B, Hq, D], scaled by 1/sqrt(D); and the planted directions [layers, B, Hkv, 1, D]."""
    g = _gen(seed, 1)
    shape = (c["layers"], c["batch"])
    x = _randn(g, *shape, c["hq"], D)
    direction = _randn(g, *shape, c["hkv"], 1, D)
    direction /= direction.norm(dim=-1, keepdim=True)
    if c["planted"]:
        m = direction.squeeze(-2).repeat_interleave(c["hq"] // c["hkv"], dim=2) * math.sqrt(D)
        x = math.sqrt(1 - PLANT_RHO ** 2) * x + PLANT_RHO * m
    return (x / math.sqrt(D)).to(torch.bfloat16), direction


def _layer_cache(c, seed, layer, seg, direction):
    """K and V of one layer in sequence order, bf16 [B, Hkv, L, D]; NaN past each sequence's current token."""
    g = _gen(seed, 2, layer)
    length = int(seg.sum(axis=1).max())
    k = _randn(g, c["batch"], c["hkv"], length, D)
    v = _randn(g, c["batch"], c["hkv"], length, D)
    pos = torch.arange(length, device="cuda").view(1, 1, -1)
    if c["planted"]:
        lo = torch.from_numpy(seg[:, 0].copy()).cuda().view(-1, 1, 1)
        hi = lo + torch.from_numpy(seg[:, 1].copy()).cuda().view(-1, 1, 1)
        hit = torch.rand(k.shape[:3], generator=g, device="cuda") < PLANT_SHARE
        k += ((pos >= lo) & (pos < hi) & hit).unsqueeze(-1) * (PLANT_LIFT / PLANT_RHO) * direction[layer]
    past = (pos >= torch.from_numpy(seg.sum(axis=1)).cuda().view(-1, 1, 1)).unsqueeze(-1)
    nan = torch.tensor(float("nan"), device="cuda")
    return (torch.where(past, nan, k).to(torch.bfloat16), torch.where(past, nan, v).to(torch.bfloat16))


def _current(x, seg):
    """The current token's rows [B, Hkv, D] of a sequence-ordered cache."""
    b = torch.arange(x.shape[0], device="cuda")
    return x[b, :, torch.from_numpy(seg.sum(axis=1) - 1).cuda()]


def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def prepare(c, seed):
    seg, pols = _layout(c)
    nl, b, hq, hkv, per = c["layers"], c["batch"], c["hq"], c["hkv"], c["per_call"]
    keep = int(_kept_counts(c).max())
    q, direction = _queries(c, seed)
    s = {"case": c, "q": q, "seg": _i32(seg), "keep": keep}
    per_layer = c["dense_layers"] > 0
    s["pol"] = _i32(np.stack(pols)) if per_layer else _i32(pols[-1])
    s["mode"] = M.MURMUR_POL_PER_SEQ | (M.MURMUR_POL_PER_LAYER if per_layer else 0)
    s["dtype"] = M.MURMUR_DTYPE_F32 if c["out_f32"] else M.MURMUR_DTYPE_BF16
    s["out"] = torch.zeros((nl, b, hq, D), dtype=torch.float32 if c["out_f32"] else torch.bfloat16, device="cuda")
    s["lse"] = torch.zeros((nl, b, hq), dtype=torch.float32, device="cuda")
    s["ws_bytes"] = M.murmur_decode_attn_workspace(per, b, hq, hkv, keep, 0)
    s["ws"] = torch.zeros(s["ws_bytes"] // 4 + 64, dtype=torch.int32, device="cuda")
    sets = (nl if per_layer else 1) * b
    s["idx"] = torch.full((sets, keep), -1, dtype=torch.int32, device="cuda")
    s["count"] = torch.zeros(sets, dtype=torch.int32, device="cuda")
    s["ranges"] = torch.zeros((sets, M.N_PIECES, 2), dtype=torch.int32, device="cuda")

    # where each cache row's token lies in sequence order (-1: no token)
    total = seg.sum(axis=1)
    if c["api"] == "ring":
        out0 = total - seg[:, 3]
        rows = int(-(-(out0.max() + c["sink_o"] + c["w_o"]) // 8) * 8)
        source = np.full((b, rows), -1, dtype=np.int64)
        for i in range(b):
            source[i, :out0[i]] = np.arange(out0[i])
            before = int(seg[i, 3]) - 1  # the current token is appended by the step itself
            tok = np.concatenate([np.arange(min(c["sink_o"], before)),
                                  np.arange(max(c["sink_o"], before - c["w_o"]), before)]).astype(np.int64)
            at = np.where(tok < c["sink_o"], tok, c["sink_o"] + (tok - c["sink_o"]) % c["w_o"])
            source[i, out0[i] + at] = out0[i] + tok
        shape = (nl, b, hkv, rows, D)
    elif c["api"] == "paged":
        bs = c["block"]
        blocks = -(-total // bs)
        rng = np.random.default_rng(seed)
        n_blocks = int(blocks.sum()) + 8
        perm = rng.permutation(n_blocks).astype(np.int32)
        table = np.full((b, int(blocks.max())), -1, dtype=np.int32)
        source = np.full((n_blocks * bs, 2), -1, dtype=np.int64)
        at = 0
        for i in range(b):
            held = -(-(int(total[i]) - 1) // bs)  # a new block for the current token comes from the free stack
            table[i, :held] = perm[at:at + held]
            at += held
            p = np.arange(int(total[i]) - 1)
            r = table[i, p // bs].astype(np.int64) * bs + p % bs
            source[r, 0], source[r, 1] = i, p
        free = np.zeros(n_blocks, dtype=np.int32)
        free[:n_blocks - at] = perm[at:]
        s.update(table=_i32(table), stack=_i32(free), top=_i32([n_blocks - at]), blocks=table.shape[1],
                 n_blocks=n_blocks)
        shape = (nl, n_blocks * bs, hkv, D)
    else:
        shape = (nl, b, hkv, int(-(-total.max() // 8) * 8), D)

    k = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    if c["api"] in ("ring", "paged"):
        s["k_new"] = torch.empty((nl, b, hkv, D), dtype=torch.bfloat16, device="cuda")
        s["v_new"] = torch.empty_like(s["k_new"])
    for layer in range(nl):
        for dst, new, x in zip((k, v), ("k_new", "v_new"), _layer_cache(c, seed, layer, seg, direction)):
            if c["api"] == "ring":
                at = torch.from_numpy(source).cuda().view(b, 1, -1, 1)
                y = torch.gather(x, 2, at.clamp(min=0).expand(-1, hkv, -1, D))
                y.view(torch.int16).masked_fill_(at < 0, NAN_BITS)
                dst[layer] = y
            elif c["api"] == "paged":
                at = torch.from_numpy(source).cuda()
                y = x[at[:, 0].clamp(min=0), :, at[:, 1].clamp(min=0)]
                y.view(torch.int16).masked_fill_((at[:, :1] < 0).unsqueeze(-1), NAN_BITS)
                dst[layer] = y
            else:
                dst[layer, :, :, :x.shape[2]] = x
                dst[layer, :, :, x.shape[2]:].view(torch.int16).fill_(NAN_BITS)
            if new in s:
                s[new][layer] = _current(x, seg)
    s["k"], s["v"] = k, v

    s["calls"] = calls = []  # (first layer, murmur_kv, murmur_ring) of each attention call
    for layer in range(0, nl, per):
        if c["api"] == "paged":
            rows = shape[1]
            kv = M.make_kv(k[layer], v[layer], per, rows, (rows * hkv * D, 0, D, hkv * D))
        else:
            kv = M.kv_from_tensors(k[layer:layer + per], v[layer:layer + per])
        ring = M.make_ring(c["w_o"], s["k_new"][layer], s["v_new"][layer]) if c["api"] == "ring" else None
        calls.append((layer, kv, ring))
    if c["api"] == "paged":
        rows = shape[1]
        s["pool"] = M.make_kv(k, v, nl, rows, (rows * hkv * D, 0, D, hkv * D))
        if int(seg[:, 3].min()) > 1:  # the steps before this one: what left the windows is free already
            before = seg.copy()
            before[:, 3] -= 1
            M.murmur_paged_step(_i32(before), s["pol"], s["mode"], b, s["table"], s["blocks"], c["block"],
                                s["stack"], s["top"], s["n_blocks"], full_scan=True)
    if c["graph"]:
        keep_state = [s[n].clone() for n in ("table", "stack", "top") if n in s]
        _token(s)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _token(s)
        for n, x in zip(("table", "stack", "top"), keep_state):
            s[n].copy_(x)
        s["graph"] = graph
    return s


# ---- one token ------------------------------------------------------------------------------------------------------

def _token(s):
    """Every call of one generated token, on the current stream."""
    c = s["case"]
    b, hq, hkv, per, keep = c["batch"], c["hq"], c["hkv"], c["per_call"], s["keep"]
    api, out, lse, q = c["api"], s["out"], s["lse"], s["q"]
    if api == "paged":
        M.murmur_paged_step(s["seg"], s["pol"], s["mode"], b, s["table"], s["blocks"], c["block"], s["stack"],
                            s["top"], s["n_blocks"], False, s["pool"], hkv, s["k_new"], s["v_new"])
        M.murmur_evict_compact_paged(s["seg"], s["pol"], s["mode"], b, s["table"], s["blocks"], c["block"], s["idx"],
                                     keep, s["count"])
    elif api in ("ranges", "index"):
        M.murmur_evict_compact(s["seg"], s["pol"], s["mode"], b, s["idx"], keep, s["count"], s["ranges"])
    for layer, kv, ring in s["calls"]:
        lists = (s["idx"], s["count"], s["ranges"]) if c["lists"] else (None, None, None)
        rest = (keep, b, hq, hkv, D, 1.0, 0, out[layer], s["dtype"], lse[layer], s["ws"], s["ws_bytes"])
        if api == "step":
            M.murmur_decode_step(s["seg"], s["pol"], s["mode"], q[layer], kv, *lists, *rest)
        elif api == "ring":
            M.murmur_decode_step_ring(s["seg"], s["pol"], s["mode"], ring, q[layer], kv, None, None, None, *rest)
        elif api == "ranges":
            M.murmur_decode_attn(q[layer], kv, None, s["ranges"], None, *rest)
        else:
            M.murmur_decode_attn(q[layer], kv, s["idx"], None, s["count"], *rest)


def run(s):
    if "graph" in s:
        s["graph"].replay()
    else:
        _token(s)
    c = s["case"]
    got = [s["out"], s["lse"]]
    if c["lists"] or c["api"] in ("ranges", "index"):
        got += [s["idx"], s["count"], s["ranges"]]
    if c["api"] == "paged":
        got += [s["idx"], s["count"], s["table"], s["stack"], s["top"], s["k"], s["v"]]
    if c["api"] == "ring":
        got += [s["k"], s["v"]]
    return got


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def exact(c, seed):
    seg, pols = _layout(c)
    q, direction = _queries(c, seed)
    nl, b, hq, hkv = c["layers"], c["batch"], c["hq"], c["hkv"]
    out = torch.empty((nl, b, hq, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((nl, b, hq), dtype=torch.float64, device="cuda")
    kept = {}
    for layer in range(nl):
        k, v = _layer_cache(c, seed, layer, seg, direction)
        for i in range(b):
            key = (i, id(pols[layer]))
            if key not in kept:
                kept[key] = torch.from_numpy(_kept(seg[i], pols[layer][i])).cuda()
            for g in range(hkv):
                kk, vv = (x[i, g].index_select(0, kept[key]).double() for x in (k, v))
                heads = slice(g * (hq // hkv), (g + 1) * (hq // hkv))
                logits = q[layer, i, heads].double() @ kk.t().contiguous()
                lse[layer, i, heads] = torch.logsumexp(logits, dim=-1)
                out[layer, i, heads] = torch.softmax(logits, dim=-1) @ vv
    return [out, lse] + [None] * {"ring": 2, "paged": 7}.get(c["api"], 0 if c["api"] == "step" and not c["lists"] else 3)

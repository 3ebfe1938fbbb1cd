"""The work this library is timed on: decoding, the periodic schedule and prompt eviction, through its
public entry points, over the shapes that its configurations and tests span.

A case is a plain dict.  Fields:
  kind     "decode": `tokens` new tokens per sequence, each through `layers` layers, one eviction per token
           "periodic": `tau` tokens that only attend, each through `layers` layers, then one compression event
           "prompt": one layer takes a whole prompt of `context` tokens and evicts it to `budget`
           "chunk": one layer holding `budget` entries takes `context` further prompt tokens, evicts to `budget`
  batch, n_q_heads, n_kv_heads, budget, n_recent: the layer's shape (head_dim 128, n_q_heads / 4 indexer heads)
  shared   the head-shared layout (one indexer key, eviction set and memory per sequence)
  path     how a decode token runs: "fused" (im_decode_step), "group" (index reuse: the first layer of every four
           decides, the others follow its slot), "steps" (the six separate calls)
  graph    the decode tokens are replayed from a captured HIP graph instead of being launched one by one
  dist     distribution of the keys (workloads/synth.py)

Caches of several layers exceed the last-level cache together, as a model's do.
"""
from __future__ import annotations

import math

import torch

import paper_2605_25475_amd as im
from workloads import Workload, hidden_stream, layer_params, token_stream

DEV = "cuda"
DEFAULTS = dict(kind="decode", batch=1, n_q_heads=32, n_kv_heads=8, context=0, budget=256, n_recent=0, layers=1,
                tokens=1, tau=0, shared=False, path="fused", graph=False, dist="normal")


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # one layer, one token, batch 1: what a single small call costs (launches and latency)
        _case("decode-b1-256", budget=256),
        # decoding at the 16K-context shape the headline figure is quoted on: replayed from a graph, as in serving
        _case("decode-b4-2048-graph", batch=4, budget=2048, layers=8, tokens=4, graph=True, dist="mixture"),
        # many sequences, a small budget, 7 query heads per KV head; launched token by token
        _case("decode-b16-512-g7", batch=16, n_q_heads=28, n_kv_heads=4, budget=512, layers=8, tokens=4, dist="planted"),
        # one long sequence with a large budget
        _case("decode-b1-4096", budget=4096, layers=8, tokens=4, dist="walk"),
        # index reuse over groups of four layers: two leaders, six followers
        _case("decode-b8-1024-group", batch=8, budget=1024, layers=8, tokens=4, path="group", dist="planted"),
        # the layer-wide layout of the method's text
        _case("decode-b4-2048-shared", batch=4, budget=2048, layers=8, tokens=4, shared=True, dist="mixture"),
        # the separate calls, as a program uses that looks at scores and lists between them; ragged sizes
        _case("decode-b3-777-steps", batch=3, n_q_heads=24, n_kv_heads=8, budget=777, n_recent=32, layers=4,
              tokens=2, path="steps"),
        # the periodic schedule: attention for 128 tokens, then one compression event
        _case("periodic-b4-2048-128", kind="periodic", batch=4, budget=2048, layers=2, tau=128, dist="mixture"),
        # prompt eviction at the 16K-context shape
        _case("prompt-b4-16384", kind="prompt", batch=4, context=16384, budget=2048, dist="mixture"),
        # one chunk of a 128K-token prompt on top of the running cache
        _case("chunk-b1-4096", kind="chunk", context=4096, budget=4096, dist="walk"),
        # prompt eviction of a batch in the layer-wide layout
        _case("prompt-b8-4096-shared", kind="prompt", batch=8, context=4096, budget=1024, shared=True, dist="planted"),
        # a short prompt of odd length
        _case("prompt-b2-1500", kind="prompt", batch=2, n_q_heads=28, n_kv_heads=4, context=1500, budget=333,
              n_recent=7),
    ]


HEADS = [(32, 8), (28, 4), (24, 8), (40, 8), (16, 4), (64, 8), (8, 8)]


def _log(rng, lo, hi):
    """A whole number, uniform in its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "periodic", "prompt", "prompt", "chunk"])
    hq, hk = rng.choice(HEADS)
    shared = rng.random() < 0.3
    dist = rng.choice(["normal", "planted", "mixture", "walk"])
    c = _case(kind=kind, n_q_heads=hq, n_kv_heads=hk, shared=shared, dist=dist, batch=_log(rng, 1, 16),
              n_recent=rng.choice([0, 0, rng.randint(1, 32)]))
    slots = 65536   # batch x KV heads x entries of the largest listed cache
    if kind in ("decode", "periodic"):
        c["budget"] = _log(rng, 64, min(4096, slots // (c["batch"] * hk)))
        if kind == "decode":
            c["path"] = rng.choice(["fused", "fused", "group", "steps"])
            c["layers"], c["tokens"] = rng.randint(1, 8), rng.randint(1, 4)
            c["graph"] = c["path"] == "fused" and rng.random() < 0.4
        else:
            c["layers"], c["tau"] = rng.randint(1, 2), rng.randint(16, 128)
    elif kind == "prompt":
        # (the largest listed prompt: 4 sequences of 16384 tokens, 32 heads)
        c["batch"] = _log(rng, 1, 8)
        most = min(16384, 65536 // c["batch"], int(math.sqrt(4 * 8 * 16384 ** 2 * 32 / (c["batch"] * hk * hq))))
        c["context"] = _log(rng, 300, most)
        c["budget"] = max(c["n_recent"] + 4, int(c["context"] * rng.uniform(0.03, 0.5)))
    else:
        c["batch"] = _log(rng, 1, 4)
        c["context"], c["budget"] = _log(rng, 256, 4096), _log(rng, 256, 4096)
    return c


def _workload(c, seed, context):
    return Workload("case", 1000 + seed, c["n_q_heads"], c["n_kv_heads"], c["layers"], c["batch"], context, c["budget"],
                    c["tokens"], c["dist"], planted_frac=0.05, head_shared=c["shared"], n_recent=c["n_recent"],
                    idx_dim=16 if c["shared"] else 64)


def _layer(c, w, handle, li, n_tokens):
    """One layer with its weights, and its first n_tokens tokens: (layer, K, V, Q, X)."""
    p = layer_params(w, li, DEV)
    params = im.Params(p["Uq"], p["G"], p["Uk"], p["Wtheta"], p["wg"], p["cg"], p["norm_q_w"], p["norm_k_w"])
    K, V, Q = token_stream(w, li, DEV, n_tokens=n_tokens)
    X = hidden_stream(w, li, DEV, n_tokens=n_tokens) if c["shared"] else Q.view(w.batch, n_tokens, -1)
    return im.Layer(handle, params, DEV), K, V, Q, X


def _handle(c, w, capacity, max_queries):
    return im.Handle(im.Config(batch=w.batch, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, capacity=capacity,
                               n_idx_heads=w.n_idx_heads, idx_dim=w.idx_dim, n_sink=w.n_sink, n_recent=w.n_recent,
                               fold_block=w.fold_block, max_queries=max_queries, head_shared=int(w.head_shared)), DEV)


def _positions(w, t0, t1):
    return torch.arange(t0, t1, dtype=torch.int32, device=DEV).repeat(w.batch, 1).contiguous()


def _append(c, layer, k, v, x, pos):
    if c["shared"]:
        im.im_append_kv_hidden(layer.h, layer.p, layer.st, k, v, x, pos)
    else:
        im.im_append_kv(layer.h, layer.st, k, v, pos)


def _kept(layer, n):
    """What a layer holds after an eviction to n entries (views of its state)."""
    st = layer.st
    return {"K": st.K[:, :, :n], "V": st.V[:, :, :n], "Kidx": st.Kidx[..., :n, :], "pos": st.pos[..., :n],
            "len": st.len, "M": st.M, "b": st.b}


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    return {"decode": _prepare_decode, "periodic": _prepare_decode, "prompt": _prepare_prompt,
            "chunk": _prepare_prompt}[c["kind"]](c, seed)


def _prepare_decode(c, seed):
    """Layers in the steady state of decoding: a prompt a quarter longer than the budget has been evicted to it
    (scored by its last 64 queries), the memory holds what left, and the next tokens' q, k, v are at hand."""
    B, n_new = c["batch"], c["tau"] if c["kind"] == "periodic" else c["tokens"]
    L = c["budget"] + max(16, c["budget"] // 4)
    w = _workload(c, seed, L)
    nw = min(64, L)
    s = {"c": c, "w": w, "layers": [], "in": []}
    s["handle"] = h = _handle(c, w, max(L, c["budget"] + max(1, c["tau"])), max(nw, n_new))
    for li in range(c["layers"]):
        layer, K, V, Q, X = _layer(c, w, h, li, L + n_new)
        cut = lambda t: t.contiguous()
        im.im_set_max_live(h, L)
        lead = s["layers"][li - li % 4] if c["path"] == "group" and li % 4 else None
        _append(c, layer, cut(K[:, :, :L]), cut(V[:, :, :L]), cut(X[:, :L]), _positions(w, 0, L))
        if lead is None:
            layer.compress(cut(Q[:, L - nw:L]), cut(X[:, L - nw:L]), _positions(w, L - nw, L), c["budget"], w.lam, w.eta)
        else:   # a follower's slots are its leader's
            im.im_memory_update(h, layer.p, layer.st, lead.evict_idx, lead.n_evict, w.lam, w.eta)
            im.im_compact_kv(h, layer.st, lead.keep_idx, lead.n_keep, lead.evict_idx, lead.n_evict)
        s["layers"].append(layer)
        s["in"].append([(cut(K[:, :, L + t:L + t + 1]), cut(V[:, :, L + t:L + t + 1]), cut(Q[:, L + t]), cut(X[:, L + t]))
                        for t in range(n_new)])
        if c["kind"] == "periodic":
            s.setdefault("window", []).append((cut(Q[:, L:]), cut(X[:, L:])))
    im.im_set_max_live(h, c["budget"] + max(1, c["tau"]))
    s["pos"] = [_positions(w, L + t, L + t + 1) for t in range(n_new)]
    s["pos_window"] = _positions(w, L, L + n_new)
    s["out"] = torch.empty((n_new, c["layers"], B, w.n_q_heads, 128), dtype=torch.bfloat16, device=DEV)
    s["evicted"] = torch.full((c["tokens"], c["layers"]) + tuple(h.cfg.set_shape()), -1, dtype=torch.int32, device=DEV)
    s["outputs"] = {"out": s["out"], "evicted": s["evicted"], "layers": [_kept(la, c["budget"]) for la in s["layers"]]}
    assert im.im_query_status(h) == 0
    if c["graph"]:
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _decode(s)
    return s


def _prepare_prompt(c, seed):
    """A prompt's (or a chunk's) q, k, v as the projections leave them, and the layer that takes them."""
    L = c["context"]
    held = c["budget"] if c["kind"] == "chunk" else 0
    w = _workload(c, seed, held + L)
    s = {"c": c, "w": w}
    s["handle"] = h = _handle(c, w, held + L, L)
    layer, K, V, Q, X = _layer(c, w, h, 0, held + L)
    if held:
        _append(c, layer, K[:, :, :held].contiguous(), V[:, :, :held].contiguous(), X[:, :held].contiguous(),
                _positions(w, 0, held))
        layer.compress(Q[:, :held][:, :64].contiguous(), X[:, :held][:, :64].contiguous(), _positions(w, 0, min(64, held)),
                       c["budget"], w.lam, w.eta)   # nothing leaves: the held entries get their indexer keys
    s["layer"] = layer
    s["k"], s["v"] = K[:, :, held:].contiguous(), V[:, :, held:].contiguous()
    s["q"], s["x"] = Q[:, held:].contiguous(), X[:, held:].contiguous()
    s["pos"] = _positions(w, held, held + L)
    s["q_last"] = s["q"][:, -1].contiguous()
    n, keep = held + L, c["budget"]
    s["outputs"] = {"out": layer.out, "scores": layer.scores[..., :n], "keep": layer.keep_idx[..., :keep],
                    "evict": layer.evict_idx[..., :n - keep], "n_keep": layer.n_keep, "n_evict": layer.n_evict,
                    **_kept(layer, keep)}
    assert im.im_query_status(h) == 0
    return s


def _decode(s):
    c, w = s["c"], s["w"]
    h, B = s["handle"], c["batch"]
    for t in range(c["tokens"]):
        pos = s["pos"][t]
        p1 = pos.view(B)
        for li, layer in enumerate(s["layers"]):
            k, v, q, x = s["in"][li][t]
            out, evicted = s["out"][t, li], s["evicted"][t, li]
            if c["path"] == "steps":
                layer.step(k, v, pos, q.unsqueeze(1), x.unsqueeze(1), pos, q, c["budget"], w.lam, w.eta,
                           x_new=x.unsqueeze(1))
                out.copy_(layer.out)
            elif c["path"] == "group" and li % 4:
                slot = s["evicted"][t, li - li % 4]
                if c["shared"]:
                    im.im_decode_step_shared_hidden(h, layer.p, layer.st, q, x, k, v, p1, slot, w.lam, w.eta, out)
                else:
                    im.im_decode_step_shared(h, layer.p, layer.st, q, k, v, p1, slot, w.lam, w.eta, out)
            else:
                im.im_decode_step(h, layer.p, layer.st, q, x, p1, k, v, p1, c["budget"], w.lam, w.eta, out, None, evicted)


def _periodic(s):
    c, w = s["c"], s["w"]
    h, B = s["handle"], c["batch"]
    for t in range(c["tau"]):
        p1 = s["pos"][t].view(B)
        for li, layer in enumerate(s["layers"]):
            k, v, q, x = s["in"][li][t]
            if c["shared"]:
                im.im_attend_step_hidden(h, layer.p, layer.st, q, x, k, v, p1, s["out"][t, li])
            else:
                im.im_attend_step(h, layer.p, layer.st, q, k, v, p1, s["out"][t, li])
    for layer, (q, x) in zip(s["layers"], s["window"]):
        layer.compress(q, x, s["pos_window"], c["budget"], w.lam, w.eta)


def _prompt(s):
    c, w, layer = s["c"], s["w"], s["layer"]
    if c["kind"] == "prompt":   # a new sequence: the layer starts empty
        for t in (layer.st.len, layer.st.n_projected, layer.st.M, layer.st.b):
            t.zero_()
    layer.step(s["k"], s["v"], s["pos"], s["q"], s["x"], s["pos"], s["q_last"], c["budget"], w.lam, w.eta, x_new=s["x"])


def run(state):
    kind = state["c"]["kind"]
    if "graph" in state:
        state["graph"].replay()
    elif kind == "decode":
        _decode(state)
    elif kind == "periodic":
        _periodic(state)
    else:
        _prompt(state)
    return state["outputs"]


def _attend_work(c, n):
    """Bytes and operations of attending to n entries per unit with one query per sequence, readout included."""
    B, H, Hk = c["batch"], c["n_q_heads"], c["n_kv_heads"]
    units, sets = B * Hk, B if c["shared"] else B * Hk
    by = units * n * 512 + sets * (128 * 129) * 4 + B * H * 128 * 4 + 2 * 128 * 128
    fl = B * H * n * 128 * 4 + B * H * 128 * 128 * 4
    return by, fl


def work(case):
    """Every input read once, every output written once: cached rows, new rows, weights, memory states, scores."""
    c = dict(DEFAULTS, **case)
    B, H, Hk, budget = c["batch"], c["n_q_heads"], c["n_kv_heads"], c["budget"]
    Hi, di = H // 4, 16 if c["shared"] else 64
    units, sets = B * Hk, B if c["shared"] else B * Hk
    d_model = H * 128
    weights = 2 * (Hi * di + Hi) * d_model + 2 * di * (d_model if c["shared"] else 128) + 2 * 128 * 128
    memory = sets * 2 * 4 * 128 * 129        # read and written back
    row = 512                                # one K row and one V row

    def score(n_q, n, pairs):                # n cached keys per set, `pairs` visible (query, key) pairs per set
        by = B * n_q * d_model * 2 * (2 if c["shared"] else 1) + sets * n * (2 * di + 4 + 4) + weights
        return by, B * n_q * d_model * 2 * (Hi * di + Hi) + sets * pairs * Hi * di * 2

    def project(n_new):
        if c["shared"]:
            return B * n_new * (d_model * 2 + 2 * di), B * n_new * d_model * di * 2
        return units * n_new * (256 + 2 * di), units * n_new * 128 * di * 2

    def evict(n, n_out):                     # selection, memory write, compaction (at most min(n_out, budget) rows move)
        moved = min(n_out, budget, max(0, n - budget))
        by = sets * n * (8 + 4) + units * n_out * row + memory + units * moved * 2 * row
        return by, sets * n_out * 128 * 128 * 2 * 2

    total = [0.0, 0.0]

    def add(times, *parts):
        for by, fl in parts:
            total[0] += times * by
            total[1] += times * fl

    if c["kind"] == "decode":
        lead = c["layers"] if c["path"] != "group" else (c["layers"] + 3) // 4
        add(c["tokens"] * c["layers"], (2 * units * row, 0), project(1), _attend_work(c, budget), (memory / 2, 0))
        add(c["tokens"] * lead, score(1, budget + 1, budget + 1))
        add(c["tokens"] * c["layers"], (units * 3 * row, sets * 128 * 128 * 4))
    elif c["kind"] == "periodic":
        n = budget + c["tau"]
        add(c["tau"] * c["layers"], (2 * units * row, 0), project(1), _attend_work(c, budget + c["tau"] / 2))
        add(c["layers"], score(c["tau"], n, c["tau"] * (budget + c["tau"] / 2)), evict(n, c["tau"]))
    else:
        L, held = c["context"], budget if c["kind"] == "chunk" else 0
        n = L + held
        add(1, (2 * units * L * row, 0), project(L), score(L, n, L * (held + L / 2)), evict(n, n - budget),
            _attend_work(c, budget))
    return {"bytes": total[0], "flops": total[1]}


def tolerance(case):
    # Scores, lists, positions, lengths and moved rows are whole numbers or come out bit for bit; the memory state
    # and the attention output are fp32 sums (measured with the sums in another order: 3e-8 of the memory state).
    # The output is rounded to bf16 once, and another order moves a value across a rounding boundary now and
    # then: 1e-4 of the output against its 64-bit value rounded to bf16, single values by one bf16 step (0.0078).
    return {"rel": 4e-4, "max": 1.6e-2}

"""What is timed when this framework's speed is compared between two builds.

Every case is work that a decode loop has the library do through its public entry points, on the
shapes of the repository's own workloads (workloads/gen.py: a tiny fp32 round and the 4B-, 8B- and
32B-like ones) or generic ones near them.  `listed()` names twelve, `draw(rng)` gives further ones
of the same ranges: batches of 1 to 64 sequences, contexts of 64 to 32768 entries, contiguous and
paged caches, chains and trees, both head dimensions, odd vocabularies and row counts.

A case is a dict of plain values; `kind` says which calls make up one pass:
  round   k draft steps, verification attention, LM head, acceptance, replayed from a HIP graph
  close   acceptance + exit rule and the cache compaction that close a round, from a HIP graph
  draft   one specexit_draft_step
  level   one specexit_draft_tree_level (W nodes of one level, ranked continuations)
  verify  specexit_verify_attn; with layers > 1 one call per layer, replayed from a HIP graph
  head    specexit_lmhead_argmax
"""
from __future__ import annotations

import math
import random

import torch

EPS, THETA = 1e-6, 1e6
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------------------------ the cases

def _dims(D, Hq, Hkv, d, I, V):
    return {"D": D, "Hq": Hq, "Hkv": Hkv, "d": d, "I": I, "V": V}


TINY = _dims(512, 8, 2, 64, 2048, 4096)
SMALL = _dims(2048, 32, 8, 64, 8192, 128259)
L4B = _dims(2560, 32, 8, 128, 9728, 151936)
L8B = _dims(4096, 32, 8, 128, 12288, 151936)
L32B = _dims(5120, 64, 8, 128, 25600, 151936)


def _cache(lo, hi, paged=False, page=16):
    return {"lo": lo, "hi": hi, "paged": paged, "page": page}


def listed():
    return [
        # the smallest call: what closes a round of four sequences with a 16-node tree, all layers of an 8B-like cache
        {"name": "close_tree_36_layers", "kind": "close", "dtype": "bf16", "B": 4, "n_q": 16, "tree": True, "layers": 36,
         **L8B, **_cache(500, 1000)},
        # a whole round of the tiny fp32 workload: some seventy short launches, latency and nothing else
        {"name": "round_tiny_f32", "kind": "round", "dtype": "f32", "B": 1, "k": 4, **TINY, **_cache(256, 256)},
        # a whole round of one sequence on the 4B-like model: the latency-critical single-user case
        {"name": "round_4b", "kind": "round", "dtype": "bf16", "B": 1, "k": 6, **L4B, **_cache(4096, 4096)},
        # the target's 36 verification attentions of that round: short calls, one per layer
        {"name": "verify_4b_36_layers", "kind": "verify", "dtype": "bf16", "B": 1, "n_q": 7, "tree": False, "layers": 36,
         **L4B, **_cache(4096, 4096)},
        # tree verification with 64-wide heads over a paged cache with larger pages
        {"name": "verify_d64_tree", "kind": "verify", "dtype": "bf16", "B": 8, "n_q": 16, "tree": True, "layers": 1,
         **SMALL, **_cache(1000, 8000, True, 32)},
        # long-context verification of a batch (the largest workload)
        {"name": "verify_32b_long", "kind": "verify", "dtype": "bf16", "B": 16, "n_q": 9, "tree": False, "layers": 1,
         **L32B, **_cache(8192, 32768, True)},
        # draft steps: an ordinary batch, the largest workload, the most sequences a step takes
        {"name": "draft_8b_batch8", "kind": "draft", "dtype": "bf16", "B": 8, **L8B, **_cache(2048, 16384, True)},
        {"name": "draft_32b_long", "kind": "draft", "dtype": "bf16", "B": 16, **L32B, **_cache(8192, 32768, True)},
        {"name": "draft_8b_batch64", "kind": "draft", "dtype": "bf16", "B": 64, **L8B, **_cache(512, 4096, True)},
        # one level of tree drafting: four sequences, four nodes each, three ranked continuations
        {"name": "level_8b_tree", "kind": "level", "dtype": "bf16", "B": 4, "W": 4, "level": 3, "top_b": 3, **L8B, **_cache(8192, 8192)},
        # LM head: the largest block, and an odd one of three sequences over a widened head
        {"name": "head_32b_rows144", "kind": "head", "dtype": "bf16", "M": 144, "n_extra": 0, **L32B},
        {"name": "head_8b_rows21", "kind": "head", "dtype": "bf16", "M": 21, "n_extra": 3, **L8B},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choices(["draft", "level", "verify", "head", "round", "close"], [6, 3, 6, 5, 2, 1])[0]
    f32 = rng.random() < 0.15
    if f32:
        dims = dict(rng.choice([TINY, _dims(1024, 16, 4, 64, 3072, 4096), _dims(1024, 8, 2, 128, 2816, 4096)]))
        dims["V"] = _log_int(rng, 4096, 20000)
    else:
        dims = dict(rng.choice([SMALL, _dims(1536, 12, 4, 128, 6144, 1), L4B, L8B, L8B, L32B]))
        dims["V"] = rng.choice([151936, _log_int(rng, 32000, 151936)])
    c = {"kind": kind, "dtype": "f32" if f32 else "bf16", **dims}
    if kind == "head":
        c.update(M=_log_int(rng, 1, 24 if f32 else 144), n_extra=rng.choice([0, 3]))
        return c
    G = c["Hq"] // c["Hkv"]
    if kind == "round":
        c.update(B=1 if not f32 else rng.randint(1, 2), k=rng.randint(3, 6))
    else:
        c["B"] = _log_int(rng, 1, 8 if f32 else 16 if c["D"] == 5120 else 64)
    # contexts: a range around a length drawn over its logarithm, all caches together within about a gigabyte
    top = (16 << 20 if f32 else 1100 << 20) // (c["B"] * c["Hkv"] * c["d"] * (8 if f32 else 4))
    mid = _log_int(rng, 64, max(128, min(2048 if f32 else 20000, top)))
    paged = rng.random() < 0.6
    c.update(_cache(max(16, int(mid * 0.5)), int(mid * 1.5), paged, rng.choice([16, 16, 32, 64]) if paged else 16))
    if kind == "verify":
        most = 128 // G
        c.update(n_q=rng.randint(2, min(17, most)), tree=rng.random() < 0.4, layers=1 if c["B"] > 2 or mid > 5000 else rng.randint(8, 36))
    elif kind == "level":
        W = rng.randint(1, max(1, min(6, 64 // c["B"])))
        c.update(W=W, level=rng.randint(1, 4), top_b=rng.randint(1, 4))
    elif kind == "close":
        c.update(n_q=rng.randint(4, 17), tree=rng.random() < 0.7, layers=rng.randint(8, 48), lo=200, hi=400, paged=False, page=16, B=min(c["B"], 8))
    return c


# ------------------------------------------------------------------------------------ inputs

class _Gen:
    """Random tensors on the GPU, from the seed alone."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1_000_003 * (seed + 1) + 7919 * case["D"] + case["V"])
        self.py = random.Random(seed * 31 + case["V"])
        self.dt = DTYPES[case["dtype"]]

    def normal(self, shape, std=1.0):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=self.dt)
        return t.mul_(std) if std != 1.0 else t

    def ids(self, shape, n):
        return torch.randint(0, n, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _spread(case):
    """Context lengths of the batch: spread evenly over the case's range (the seed only permutes them)."""
    B, lo, hi = case["B"], case["lo"], case["hi"]
    return [lo + (hi - lo) * (2 * i + 1) // (2 * B) for i in range(B)]


def _lengths(case, gen):
    n = _spread(case)
    gen.py.shuffle(n)
    return n


def _kv(case, gen, L, extra):
    """One layer's caches with `extra` block entries behind each context: (k, v, page table or None)."""
    Hkv, d, ps = case["Hkv"], case["d"], case["page"]
    if not case["paged"]:
        shape = (case["B"], Hkv, max(L) + extra, d)
        return gen.normal(shape), gen.normal(shape), None
    per = [(n + extra + ps - 1) // ps for n in L]
    pool = sum(per) + max(1, sum(per) // 10)
    perm = torch.randperm(pool, generator=gen.g, device="cuda").to(torch.int32)
    table, at = torch.zeros((case["B"], max(per)), dtype=torch.int32, device="cuda"), 0
    for b, n in enumerate(per):
        table[b, :n] = perm[at:at + n]
        at += n
    shape = (pool, Hkv, ps, d)
    return gen.normal(shape), gen.normal(shape), table


def _weights(case, gen):
    D, Hq, Hkv, d, I, V = (case[n] for n in ("D", "Hq", "Hkv", "d", "I", "V"))
    shapes = {"embed": (V, D), "w_fc": (D, 2 * D), "w_q": (Hq * d, D), "w_k": (Hkv * d, D), "w_v": (Hkv * d, D), "w_o": (D, Hq * d),
              "w_gate": (I, D), "w_up": (I, D), "w_down": (D, I), "w_head": (V + 3, D)}
    w = {n: gen.normal(s, 0.02) for n, s in shapes.items()}
    w.update({n: gen.normal((D,), 0.1).add_(1.0) for n in ("ln_attn", "ln_mlp", "ln_final")})
    return w


def _parents(case):
    """The block's topology, shared by the sequences: a chain, or a binary tree numbered level by level."""
    return [-1] + [(i - 1) // 2 if case["tree"] else i - 1 for i in range(1, case["n_q"])]


def _ancestors(parents):
    m = []
    for i, p in enumerate(parents):
        m.append((1 << i) | (m[p] if p >= 0 else 0))
    return m


def _signed(words):
    return [w - (1 << 64) if w >> 63 else w for w in words]


def _level_nodes(case):
    """W nodes of a level in a tree of W nodes per level under one root: (node ids, ancestor words, block entries)."""
    W, level = case["W"], case["level"]
    parents = [-1] + [0] * W + [i - W for i in range(W + 1, W * level + 1)]
    nodes = list(range(W * (level - 1) + 1, W * level + 1)) if level else [0]
    m = _ancestors(parents)
    return nodes, [m[i] for i in nodes], max(nodes) + 1


def _accept_inputs(case, gen, target=None):
    """Block tokens against the target's: per sequence a root path of random length matches; a third of the blocks carry a
    step-split token on it.  Signals of a sequence late in its thinking."""
    B, V, py, parents = case["B"], case["V"], gen.py, _parents(case)
    n_q = case["n_q"]
    split = sorted(py.sample(range(V - 1), 8))
    am = [[py.randrange(V - 1) for _ in range(n_q)] for _ in range(B)] if target is None else target
    tok = [[py.randrange(V - 1) for _ in range(n_q)] for _ in range(B)]
    for b in range(B):
        cur = 0
        for step in range(min(int(py.expovariate(0.3)), n_q - 1)):
            kids = [c for c in range(1, n_q) if parents[c] == cur]
            if not kids:
                break
            c = py.choice(kids)
            if target is None and py.random() < 0.1:
                am[b][cur] = py.choice(split)
            tok[b][c] = am[b][cur]
            cur = c
    sig = torch.tensor([[py.uniform(0.7, 1.0), py.uniform(0.2, 1.0), py.uniform(20.0, 400.0)] for _ in range(B)], device="cuda")
    return {"tok": _i32(tok), "am": _i32(am), "sig": sig, "split": _i32(split),
            "parent": _i32([parents] * B) if case["tree"] else None, "stop": V - 1}


def _inputs(case, seed):
    """Everything of a case that is drawn from the seed."""
    gen, kind, x = _Gen(case, seed), case["kind"], {}
    if kind == "head":
        x["w"] = gen.normal((case["V"] + case["n_extra"], case["D"]), 0.02)
        x["hidden"] = gen.normal((case["M"], case["D"]))
        return x
    L = x["L"] = _lengths(case, gen)
    B = case["B"]
    if kind in ("draft", "level", "round"):
        W = case.get("W", 1)
        extra = {"draft": 1, "round": case.get("k", 0) + 1, "level": W * case.get("level", 0) + 1}[kind]
        x["weights"] = _weights(case, gen)
        x["draft_kv"] = _kv(case, gen, L, extra)
        x["tok"] = gen.ids((B, W) if kind == "level" else (B,), case["V"])
        x["hidden"] = gen.normal((B, W, case["D"]) if kind == "level" else (B, case["D"]))
    if kind == "verify":
        x["kv"] = [_kv(case, gen, L, case["n_q"]) for _ in range(case["layers"])]
        x["q"] = gen.normal((case["layers"], B, case["n_q"], case["Hq"], case["d"]))
    if kind == "round":
        n_q = case["k"] + 1
        x["kv"] = [_kv(case, gen, L, n_q)]
        x["q"] = gen.normal((1, B, n_q, case["Hq"], case["d"]))
        x["block_hidden"] = gen.normal((B * n_q, case["D"]))
        x["lm"] = gen.normal((case["V"], case["D"]), 0.02)
        # the target prefers a known token at every block position
        want = gen.py.sample(range(case["V"] - 1), B * n_q)
        x["lm"][torch.tensor(want, device="cuda")] += (x["block_hidden"].float() * (8.0 / case["D"])).to(gen.dt)
        target = [want[b * n_q:(b + 1) * n_q] for b in range(B)]
        x["accept"] = _accept_inputs({**case, "n_q": n_q, "tree": False}, gen, target)
    if kind == "close":
        shape = (case["layers"], B, case["Hkv"], max(L) + case["n_q"], case["d"])
        x["k"], x["v"] = gen.normal(shape), gen.normal(shape)
        x["block_hidden"] = gen.normal((B, case["n_q"], case["D"]))
        x["accept"] = _accept_inputs(case, gen)
    return x


# ------------------------------------------------------------------------------------ prepare and run

class _Graph:
    """A recorded sequence of calls, released with its owner."""

    def __init__(self, sx, calls):
        self.sx = sx
        calls()                              # first calls set kernel attributes, which a capture forbids
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            sx.specexit_graph_begin(stream)
            try:
                calls()
            finally:
                self.handle = sx.specexit_graph_end(stream)
        torch.cuda.synchronize()

    def launch(self):
        self.sx.specexit_graph_launch(self.handle)

    def __del__(self):
        self.sx.specexit_graph_destroy(self.handle)


def _buf(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _workspace(sx, nbytes, prepared=False):
    t = torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")
    if prepared:
        sx.specexit_workspace_prepare(t)
    return t


def _code(sx, case):
    return sx.BF16 if case["dtype"] == "bf16" else sx.F32


def _draft_model(sx, case, x, s):
    s["w"] = sx.draft_weights(x["weights"])
    s["dview"] = sx.kv_view(*x["draft_kv"])
    s["desc"] = sx.model_desc(_code(sx, case), *(case[n] for n in ("D", "Hq", "Hkv", "d", "I", "V")), EPS, THETA)


def _accept_state(case, x, s):
    B, n_q = case["B"], x["accept"]["tok"].shape[1]
    for n in ("accept_len", "recover", "last_node", "exit_flag", "new_ctx", "n_obs"):
        s[n] = _buf(B, torch.int32)
    s["thinking"] = _buf(B, torch.int32).fill_(1)
    s["ewma"] = _buf((B, 3), torch.float32)
    s["accept_path"] = _buf((B, n_q), torch.int32)


def _accept_call(sx, case, x, s, am, sig):
    a = x["accept"]
    sx.specexit_accept_exit(s["cfg"], case["B"], a["tok"].shape[1], a["tok"], a["parent"], am, sig, s["ctx"], a["split"], 8, s["ewma"], s["n_obs"],
                            s["thinking"], None, s["accept_len"], s["accept_path"], s["recover"], s["last_node"], s["exit_flag"], s["new_ctx"])


ACCEPT_OUT = ("accept_len", "accept_path", "recover", "last_node", "exit_flag", "new_ctx", "n_obs", "thinking", "ewma")


def prepare(case, seed):
    from paper_2509_24248_amd import binding as sx
    kind, x = case["kind"], _inputs(case, seed)
    dt, f32, i32 = DTYPES[case["dtype"]], torch.float32, torch.int32
    s = {"case": case, "sx": sx, "x": x}
    if kind == "head":
        M, V, n = case["M"], case["V"], case["n_extra"]
        s["out"] = {"argmax": _buf(M, i32), "max_logit": _buf(M, f32), "extra": _buf((M, n), f32) if n else None}
        s["ws"] = _workspace(sx, sx.specexit_lmhead_argmax_workspace_bytes(_code(sx, case), M, case["D"], V, n))
        return s
    B, L = case["B"], x["L"]
    s["ctx"] = _i32(L)
    s["scale"] = case["d"] ** -0.5
    if kind == "draft":
        _draft_model(sx, case, x, s)
        s["ws"] = _workspace(sx, sx.specexit_draft_step_workspace_bytes(s["desc"], s["dview"], B), True)
        s["out"] = {"hidden": torch.empty_like(x["hidden"]), "tok": _buf(B, i32), "sig_raw": _buf((B, 3), f32), "sig": _buf((B, 3), f32)}
    elif kind == "level":
        _draft_model(sx, case, x, s)
        W, top_b = case["W"], case["top_b"]
        nodes, words, s["n_blk"] = _level_nodes(case)
        s["node"] = _i32(nodes)
        s["mask"] = torch.tensor(_signed(words), dtype=torch.int64, device="cuda")
        s["ws"] = _workspace(sx, sx.specexit_draft_tree_level_workspace_bytes(s["desc"], s["dview"], B, W, top_b), True)
        s["out"] = {"hidden": torch.empty_like(x["hidden"]), "cand": _buf((B, W, top_b), i32), "cand_logit": _buf((B, W, top_b), f32),
                    "sig_raw": _buf((B, W, 3), f32), "sig": _buf((B, W, 3), f32)}
    elif kind == "verify":
        s["views"] = [sx.kv_view(*kv) for kv in x["kv"]]
        s["mask"] = torch.tensor([_signed(_ancestors(_parents(case)))] * B, dtype=torch.int64, device="cuda") if case["tree"] else None
        s["out"] = {"attn": torch.empty_like(x["q"])}
        s["ws"] = _workspace(sx, sx.specexit_verify_attn_workspace_bytes(s["views"][0], B, case["n_q"], case["Hq"]))
        if case["layers"] > 1:
            s["graph"] = _Graph(sx, lambda: _verify_calls(s))
    elif kind == "close":
        s["view"] = sx.kv_view(x["k"][0], x["v"][0])
        s["hidden_next"] = _buf((B, case["D"]), dt)
        s["cfg"] = sx.exit_cfg(stop_think_token=x["accept"]["stop"])
        _accept_state(case, x, s)
        keep = x["k"].clone(), x["v"].clone()
        s["graph"] = _Graph(sx, lambda: _close_calls(s))
        x["k"].copy_(keep[0])
        x["v"].copy_(keep[1])
        _reset_accept(s)
    else:
        _draft_model(sx, case, x, s)
        k, n_q = case["k"], case["k"] + 1
        s["pos"] = [_i32([n + j for n in L]) for j in range(k)]
        s["views"] = [sx.kv_view(*x["kv"][0])]
        s["cfg"] = sx.exit_cfg(stop_think_token=x["accept"]["stop"])
        s["ws"] = _workspace(sx, sx.specexit_draft_step_workspace_bytes(s["desc"], s["dview"], B), True)
        s["ws_attn"] = _workspace(sx, sx.specexit_verify_attn_workspace_bytes(s["views"][0], B, n_q, case["Hq"]))
        s["ws_head"] = _workspace(sx, sx.specexit_lmhead_argmax_workspace_bytes(_code(sx, case), B * n_q, case["D"], case["V"], 0))
        s["out"] = {"hidden": _buf((k, B, case["D"]), dt), "tok": _buf((k, B), i32), "sig_raw": _buf((k, B, 3), f32), "sig": _buf((k, B, 3), f32),
                    "attn": torch.empty_like(x["q"]), "argmax": _buf((B, n_q), i32), "max_logit": _buf((B, n_q), f32)}
        _accept_state(case, x, s)
        s["graph"] = _Graph(sx, lambda: _round_calls(s))
        _reset_accept(s)
    return s


def _reset_accept(s):
    s["ewma"].zero_()
    s["n_obs"].zero_()
    s["thinking"].fill_(1)


def _verify_calls(s):
    case, x, sx = s["case"], s["x"], s["sx"]
    for l in range(case["layers"]):
        sx.specexit_verify_attn(s["views"][l], case["B"], case["n_q"], case["Hq"], x["q"][l], s["ctx"], s["mask"], s["scale"], s["out"]["attn"][l], s["ws"])


def _close_calls(s):
    case, x, sx = s["case"], s["x"], s["sx"]
    _accept_call(sx, case, x, s, x["accept"]["am"], x["accept"]["sig"])
    sx.specexit_kv_compact(s["view"], case["layers"], x["k"].stride(0) * x["k"].element_size(), case["B"], case["n_q"], s["ctx"], s["accept_path"],
                           s["accept_len"], s["last_node"], x["block_hidden"], case["D"], s["hidden_next"])


def _round_calls(s):
    case, x, sx, o = s["case"], s["x"], s["sx"], s["out"]
    B, k = case["B"], case["k"]
    tok, hidden = x["tok"], x["hidden"]
    for j in range(k):
        sx.specexit_draft_step(s["desc"], s["w"], s["dview"], B, tok, hidden, s["pos"][j], o["hidden"][j], o["tok"][j], o["sig_raw"][j], o["sig"][j], s["ws"],
                               flags=sx.FLAG_WORKSPACE_PREPARED)
        tok, hidden = o["tok"][j], o["hidden"][j]
    sx.specexit_verify_attn(s["views"][0], B, k + 1, case["Hq"], x["q"][0], s["ctx"], None, s["scale"], o["attn"][0], s["ws_attn"])
    sx.specexit_lmhead_argmax(_code(sx, case), B * (k + 1), case["D"], case["V"], 0, x["block_hidden"], x["lm"], o["argmax"], o["max_logit"],
                              workspace=s["ws_head"])
    _accept_call(sx, case, x, s, o["argmax"], o["sig"][0])


def run(state):
    s = state
    case, x, sx, kind, o = s["case"], s["x"], s["sx"], s["case"]["kind"], s.get("out")
    if kind == "head":
        sx.specexit_lmhead_argmax(_code(sx, case), case["M"], case["D"], case["V"], case["n_extra"], x["hidden"], x["w"], o["argmax"], o["max_logit"],
                                  o["extra"], workspace=s["ws"])
        return o
    if kind == "draft":
        sx.specexit_draft_step(s["desc"], s["w"], s["dview"], case["B"], x["tok"], x["hidden"], s["ctx"], o["hidden"], o["tok"], o["sig_raw"], o["sig"],
                               s["ws"], flags=sx.FLAG_WORKSPACE_PREPARED)
        return {**o, "k": x["draft_kv"][0], "v": x["draft_kv"][1]}
    if kind == "level":
        sx.specexit_draft_tree_level(s["desc"], s["w"], s["dview"], case["B"], case["W"], x["tok"], x["hidden"], s["ctx"], case["level"], s["node"],
                                     s["mask"], s["n_blk"], case["top_b"], o["hidden"], o["cand"], o["cand_logit"], o["sig_raw"], o["sig"], s["ws"],
                                     flags=sx.FLAG_WORKSPACE_PREPARED)
        return {**o, "k": x["draft_kv"][0], "v": x["draft_kv"][1]}
    if kind == "verify":
        if case["layers"] > 1:
            s["graph"].launch()
        else:
            _verify_calls(s)
        return o
    s["graph"].launch()
    accept = {n: s[n] for n in ACCEPT_OUT}
    if kind == "close":
        return {**accept, "hidden_next": s["hidden_next"], "k": x["k"], "v": x["v"]}
    return {**o, **accept, "k": x["draft_kv"][0], "v": x["draft_kv"][1]}


# ------------------------------------------------------------------------------------ the same in 64 bits

def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _lin(x, w, rows=16384):
    return torch.cat([x @ w[i:i + rows].double().t() for i in range(0, w.shape[0], rows)], -1)


def _rope(x, pos):
    """x [rows, heads, d], rotate-half pairing."""
    half = x.shape[-1] // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / x.shape[-1])
    ang = (pos.double()[:, None] * inv)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _rows_of(case, pool, table, b, n):
    """The first n entries of sequence b: [Hkv, n, d] in 64 bits."""
    if table is None:
        return pool[b, :, :n].double()
    pages = (n + case["page"] - 1) // case["page"]
    return pool[table[b, :pages].long()].double().permute(1, 0, 2, 3).reshape(case["Hkv"], -1, case["d"])[:, :n]


def _attend(case, q, k, v, L, words):
    """q [n, Hq, d] against k, v [Hkv, L + block, d]; words: visible block entries per query."""
    n, Hkv, G, d = q.shape[0], case["Hkv"], case["Hq"] // case["Hkv"], case["d"]
    qs = q.reshape(n, Hkv, G, d).permute(1, 0, 2, 3).reshape(Hkv, n * G, d).contiguous()
    s = torch.matmul(qs, k.transpose(1, 2).contiguous()) * d ** -0.5
    seen = torch.ones((n, k.shape[1]), dtype=torch.bool, device="cuda")
    seen[:, L:] = torch.tensor([[bool(w >> j & 1) for j in range(k.shape[1] - L)] for w in words], device="cuda")
    s = s.masked_fill(~seen.repeat_interleave(G, 0)[None], -math.inf)
    o = torch.matmul(torch.softmax(s, -1), v.contiguous())
    return o.reshape(Hkv, n, G, d).permute(1, 0, 2, 3).reshape(n, Hkv * G * d)


def _exact_draft(case, x, tok, hidden, L, level, nodes, words, n_blk, caches):
    """One draft forward over B * W rows; the 64-bit caches are written in place."""
    w, table = x["weights"], x["draft_kv"][2]
    B, W = case["B"], len(nodes)
    Hq, Hkv, d, V = case["Hq"], case["Hkv"], case["d"], case["V"]
    xin = torch.cat([w["embed"][tok.reshape(-1).long()].double(), hidden.reshape(B * W, -1).double()], -1)
    h = _lin(xin, w["w_fc"])
    n = _rms(h, w["ln_attn"])
    pos = torch.tensor([p + level for p in L for _ in nodes], device="cuda")
    q = _rope(_lin(n, w["w_q"]).reshape(B * W, Hq, d), pos)
    k = _rope(_lin(n, w["w_k"]).reshape(B * W, Hkv, d), pos)
    v = _lin(n, w["w_v"]).reshape(B * W, Hkv, d)
    out = []
    for b in range(B):
        for i, node in enumerate(nodes):
            p = L[b] + node
            for cache, new in zip(caches, (k, v)):
                if table is None:
                    cache[b, :, p] = new[b * W + i]
                else:
                    cache[int(table[b, p // case["page"]]), :, p % case["page"]] = new[b * W + i]
        kb, vb = (_rows_of(case, c, table, b, L[b] + n_blk) for c in caches)
        out.append(_attend(case, q[b * W:(b + 1) * W], kb, vb, L[b], words))
    a = h + _lin(torch.cat(out), w["w_o"])
    m = _rms(a, w["ln_mlp"])
    y = a + _lin(torch.nn.functional.silu(_lin(m, w["w_gate"])) * _lin(m, w["w_up"]), w["w_down"])
    z = _lin(_rms(y, w["ln_final"]), w["w_head"])
    raw = z[:, V:]
    sig = torch.cat([torch.sigmoid(raw[:, :2]), torch.expm1(raw[:, 2:]).clamp_min(0.0)], -1)
    return y, z[:, :V], raw, sig


def _exact_verify(case, x, words):
    outs = []
    for l, (k, v, table) in enumerate(x["kv"]):
        for b, n in enumerate(x["L"]):
            kb, vb = (_rows_of(case, c, table, b, n + len(words)) for c in (k, v))
            outs.append(_attend(case, x["q"][l, b].double(), kb, vb, n, words))
    return torch.stack(outs).reshape(x["q"].shape)


def exact(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    if kind == "head":
        z = _lin(x["hidden"].double(), x["w"])
        V = case["V"]
        return {"argmax": None, "max_logit": z[:, :V].max(-1).values, "extra": z[:, V:] if case["n_extra"] else None}
    if kind == "verify":
        return {"attn": _exact_verify(case, x, _ancestors(_parents(case)))}
    if kind == "close":
        return None                       # whole numbers, moved bytes, and a first observation that is its own average
    caches = [c.double() for c in x["draft_kv"][:2]]
    if kind == "draft":
        y, _, raw, sig = _exact_draft(case, x, x["tok"], x["hidden"], x["L"], 0, [0], [1], 1, caches)
        return {"hidden": y, "tok": None, "sig_raw": raw, "sig": sig, "k": caches[0], "v": caches[1]}
    if kind == "level":
        nodes, words, n_blk = _level_nodes(case)
        y, z, raw, sig = _exact_draft(case, x, x["tok"], x["hidden"], x["L"], case["level"], nodes, words, n_blk, caches)
        B, W = case["B"], case["W"]
        return {"hidden": y.reshape(B, W, -1), "cand": None, "cand_logit": z.topk(case["top_b"], -1).values.reshape(B, W, -1),
                "sig_raw": raw.reshape(B, W, 3), "sig": sig.reshape(B, W, 3), "k": caches[0], "v": caches[1]}
    tok, hidden, steps = x["tok"], x["hidden"], []
    for j in range(case["k"]):
        y, z, raw, sig = _exact_draft(case, x, tok, hidden, [n + j for n in x["L"]], 0, [0], [1], 1, caches)
        tok, hidden = z.argmax(-1), y
        steps.append((y, raw, sig))
    hid, raw, sig = (torch.stack(t) for t in zip(*steps))
    n_q = case["k"] + 1
    words = [(2 << i) - 1 for i in range(n_q)]
    top = _lin(x["block_hidden"].double(), x["lm"]).max(-1).values.reshape(case["B"], n_q)
    return {"hidden": hid, "tok": None, "sig_raw": raw, "sig": sig, "attn": _exact_verify({**case, "n_q": n_q}, x, words), "argmax": None,
            "max_logit": top, "k": caches[0], "v": caches[1], "ewma": sig[0], **{n: None for n in ACCEPT_OUT if n != "ewma"}}


# ------------------------------------------------------------------------------------ work and tolerance

def _draft_work(case, rows, keys, e):
    D, Hd, Hk, I, V = case["D"], case["Hq"] * case["d"], case["Hkv"] * case["d"], case["I"], case["V"]
    weights = 2 * D * D + D * (Hd + 2 * Hk) + Hd * D + 3 * D * I + (V + 3) * D
    return (e * weights, 2 * e * Hk * keys + 3 * e * rows * D + 28 * rows, 2 * rows * weights + 4 * case["Hq"] * case["d"] * keys * rows // case["B"])


def _verify_work(case, n_q, keys, e):
    return (2 * e * case["Hkv"] * case["d"] * keys + 2 * e * case["B"] * n_q * case["Hq"] * case["d"],
            4 * case["Hq"] * case["d"] * n_q * keys)


def _head_work(case, M, rows_w, e):
    return e * case["D"] * (rows_w + M) + 8 * M, 2 * M * case["D"] * rows_w


def work(case):
    e, kind = (2 if case["dtype"] == "bf16" else 4), case["kind"]
    if kind == "head":
        parts = [_head_work(case, case["M"], case["V"] + case["n_extra"], e)]
    else:
        L, B = _spread(case), case["B"]
        if kind == "draft":
            w, o, f = _draft_work(case, B, sum(L) + B, e)
            parts = [(w + o, f)]
        elif kind == "level":
            w, o, f = _draft_work(case, B * case["W"], sum(L) + B * (case["W"] * case["level"] + 1), e)
            parts = [(w + o, f)]
        elif kind == "verify":
            parts = [_verify_work(case, case["n_q"], sum(L) + B * case["n_q"], e)] * case["layers"]
        elif kind == "close":
            # about half of the accepted nodes of a tree move, in every layer, read and written
            moved = B * (2 if case["tree"] else 0)
            parts = [(case["layers"] * 4 * e * moved * case["Hkv"] * case["d"] + B * (2 * e * case["D"] + 12 * case["n_q"]), 0)]
        else:
            k = case["k"]
            steps = [_draft_work(case, B, sum(L) + B * (j + 1), e) for j in range(k)]
            # a step needs the token of the one before: weights beyond the last-level cache come from memory in every step
            parts = [(w if j == 0 or w > 256e6 else 0, f) for j, (w, _, f) in enumerate(steps)] + [(o, 0) for _, o, _ in steps]
            parts += [_verify_work(case, k + 1, sum(L) + B * (k + 1), e), _head_work(case, B * (k + 1), case["V"], e)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    if case["kind"] == "close":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4, "differ": 0.01}     # 32-bit sums in another order, through one layer
    if case["kind"] == "head":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}     # exact bf16 products, 32-bit sums
    # bf16 storage of q, of the attention's probabilities and of the outputs: an element may round the other way
    return {"rel": 1e-2, "max": 0.2, "differ": 0.01}

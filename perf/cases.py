"""The work that a user of the phrase-memory library has it do, as cases to measure.

Each case drives the public entry points (paper_2607_07388_amd.tfe) the way a serving or a
construction program does: tables, projections and token buffers are made once in prepare(),
run() makes one pass of calls on the current stream, exact() is the same result in 64 bits with
plain torch.  Inputs are seeded draws with the shapes of the repository's workloads: truncated
Zipf(1.1) token ids over the 151936-token vocabulary, phrase tables of the most frequent n-grams
of such a stream, value rows N(0, 0.02), hidden states N(0, 1), a N(0, 0.1) projection."""
import math

import torch

from paper_2607_07388_amd import tfe

VOCAB = 151936
FIELD = 1 << 18  # token ids fit 18 bits
# Share of the positions of such a stream whose longest match exists, and rows retained per
# position by the multi-match entry point (both within a few per cent over these tables).
HITS, RETAINED = 0.6, 0.8
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # One decode step of a batch of 64: the latency of a single small launch.
        {"name": "decode_b64", "kind": "lookup", "dtype": "bf16", "dim": 1024, "rows": 64, "ctx": 2, "steps": 1,
         "n_max": 3, "phrases": 1 << 18, "gate": "sigmoid", "multi": False},
        # A short single-sequence prompt at full precision, odd length, constant gate.
        {"name": "prompt_f32_777", "kind": "lookup", "dtype": "f32", "dim": 1024, "rows": 1, "ctx": 0, "steps": 777,
         "n_max": 3, "phrases": 1 << 17, "gate": "const", "multi": False},
        # The repository's headline: 256 stacked batch-64 decode steps against the 2^20-phrase table.
        {"name": "stacked_decode_16384", "kind": "lookup", "dtype": "bf16", "dim": 1024, "rows": 16384, "ctx": 2,
         "steps": 1, "n_max": 3, "phrases": 1 << 20, "gate": "sigmoid", "multi": False},
        # Prefill of 8 x 4096 tokens against 2-, 3- and 4-gram phrases.
        {"name": "prefill_8x4096", "kind": "lookup", "dtype": "bf16", "dim": 1024, "rows": 8, "ctx": 0, "steps": 4096,
         "n_max": 4, "phrases": 1 << 19, "gate": "sigmoid", "multi": False},
        # Ragged prefill that retains every match (length weights).
        {"name": "multi_6x1023", "kind": "lookup", "dtype": "bf16", "dim": 1024, "rows": 6, "ctx": 0, "steps": 1023,
         "n_max": 4, "phrases": 1 << 18, "gate": "sigmoid", "multi": True},
        # 32 decode steps of a batch of 64 on a table in host memory: each step's lookup, then the scored
        # prefetch of the next step's 8 candidates a row on a side stream.
        {"name": "tiered_decode_32x64", "kind": "tiered", "dtype": "bf16", "dim": 1024, "rows": 64, "calls": 32,
         "steps": 1, "phrases": 1 << 17, "cache": 1 << 13, "candidates": 8, "budget": 64},
        # Four batches of 8 x 1024 tokens in turn on a table in host memory whose cache holds a
        # thirty-second of the rows, so that each of them misses.
        {"name": "tiered_prefill_8x1024", "kind": "tiered", "dtype": "bf16", "dim": 1024, "rows": 8, "calls": 4,
         "steps": 1024, "phrases": 1 << 17, "cache": 1 << 12, "candidates": 0, "budget": 0},
        # The early-exit head for one sequence, for the batch-64 step that feeds the prefetch, and at batch 256.
        {"name": "head_b1_k16", "kind": "head", "vocab": VOCAB, "dim": 1024, "rows": 1, "k": 16},
        {"name": "head_b64_k128", "kind": "head", "vocab": VOCAB, "dim": 1024, "rows": 64, "k": 128},
        {"name": "head_b256_k64", "kind": "head", "vocab": VOCAB, "dim": 1024, "rows": 256, "k": 64},
        # Table construction: the decode table's 2-grams, and 4-grams of documents of about 1000 tokens
        # behind a stop-phrase filter.
        {"name": "ngram2_64M", "kind": "ngram", "n": 2, "tokens": 1 << 26, "doc": 0, "skip": 0, "top": 1 << 19},
        {"name": "ngram4_docs_20M", "kind": "ngram", "n": 4, "tokens": 20000003, "doc": 1000, "skip": 5000,
         "top": 1 << 18},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "multi", "tiered", "head", "head", "ngram", "ngram"])
    if kind in ("lookup", "multi"):
        dtype = rng.choice(["bf16", "bf16", "f32"])
        dim = rng.choice([512, 1024, 2048, 4096] if dtype == "bf16" else [256, 512, 1024, 2048])
        # At most the bytes of the 8 x 4096 prefill.
        most = 32768 * 2048 // (dim * (2 if dtype == "bf16" else 4))
        positions = _log(rng, 48, most)
        decode = rng.random() < 0.5
        rows = positions if decode else min(positions, rng.randint(1, 16))
        return {"kind": "lookup", "dtype": dtype, "dim": dim, "rows": rows, "ctx": rng.randint(1, 4) if decode else 0,
                "steps": 1 if decode else positions // rows, "n_max": rng.choice([2, 3, 3, 4]),
                "phrases": _log(rng, 1 << 14, (1 << 29) // (dim * (2 if dtype == "bf16" else 4))),
                "gate": rng.choice(["sigmoid", "sigmoid", "const"]), "multi": kind == "multi"}
    if kind == "tiered":
        decode = rng.random() < 0.5
        phrases = _log(rng, 1 << 14, 1 << 17)
        return {"kind": "tiered", "dtype": rng.choice(["bf16", "f32"]), "dim": 1024,
                "rows": _log(rng, 1, 64) if decode else rng.randint(1, 8),
                "calls": rng.randint(4, 32) if decode else rng.randint(1, 4),
                "steps": 1 if decode else _log(rng, 17, 1024), "phrases": phrases,
                "cache": phrases // rng.randint(4, 32), "candidates": rng.randint(1, 16) if decode else 0, "budget": rng.randint(1, 256) if decode else 0}
    if kind == "head":
        vocab = _log(rng, 8000, 151936)
        return {"kind": "head", "vocab": vocab, "dim": rng.choice([256, 512, 1024, 1024]), "rows": _log(rng, 1, 256),
                "k": _log(rng, 1, 256)}
    tokens = _log(rng, 20000, 1 << 25)
    n = rng.randint(1, 4)
    return {"kind": "ngram", "n": n, "tokens": tokens, "doc": rng.choice([0, 300, 2000]),
            "skip": rng.choice([0, rng.randint(1, 5000)]), "top": _log(rng, 1000, max(1001, tokens // 64))}


# ---- inputs ----------------------------------------------------------------------------------


def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + tag) & 0x7FFFFFFFFFFF)
    return g


def _tokens(seed, tag, count, vocab=VOCAB):
    """`count` Zipf(1.1) token ids, int32."""
    w = torch.arange(1, vocab + 1, device="cuda", dtype=torch.float64).pow_(-1.1).cumsum_(0)
    out = torch.empty(count, dtype=torch.int32, device="cuda")
    g = _gen(seed, tag)
    for at in range(0, count, 1 << 24):
        n = min(1 << 24, count - at)
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64).mul_(w[-1])
        out[at:at + n] = torch.searchsorted(w, u, right=True).clamp_(max=vocab - 1).to(torch.int32)
    return out


def _normal(seed, tag, shape, sigma, dtype):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    g = _gen(seed, tag)
    per = max(1, (1 << 26) // shape[1])
    for at in range(0, shape[0], per):
        n = min(per, shape[0] - at)
        out[at:at + n] = torch.randn((n, shape[1]), generator=g, device="cuda") * sigma
    return out


def _windows(t, n, valid):
    """Keys of the n-token windows (n <= 4) along the last axis of t, int64, -1 where a token is below 0.
    4-gram keys do not fit 63 bits: `valid` (a _Ids) numbers their last three tokens."""
    L = t.shape[-1] - n + 1
    cols = [t[..., j:j + L].long() for j in range(n)]
    bad = torch.stack([c < 0 for c in cols]).any(0)
    key = torch.zeros_like(cols[0])
    for c in cols[-3:]:
        key = key * FIELD + c.clamp(min=0)
    if n == 4:
        ids = valid(key)
        bad |= ids < 0
        key = cols[0].clamp(min=0) * (1 << 40) + ids
    return torch.where(bad, torch.full_like(key, -1), key)


class _Ids:
    """Numbers a set of keys in ascending order; -1 for a key outside it."""

    def __init__(self, keys):
        self.keys = torch.unique(keys)

    def __call__(self, keys):
        if self.keys.numel() == 0:
            return torch.full_like(keys, -1)
        at = torch.searchsorted(self.keys, keys).clamp_(max=self.keys.numel() - 1)
        return torch.where(self.keys[at] == keys, at, torch.full_like(at, -1))


def _fields(key, n, ids):
    """The tokens of n-gram keys, oldest first, [count x n] int32."""
    head = []
    if n == 4:
        head, key = [key >> 40], ids.keys[key & ((1 << 40) - 1)]
    k = min(n, 3)
    return torch.stack(head + [(key >> (18 * (k - 1 - j))) & (FIELD - 1) for j in range(k)], -1).to(torch.int32)


def _phrases(seed, count, n_max):
    """The most frequent 2- to n_max-grams of a seeded stream, an equal number of each length, most
    frequent first: tokens [P x n_max] and lengths [P]."""
    stream = _tokens(seed, 1, max(1 << 17, 8 * count))
    toks, lens, cnts = [], [], []
    for n in range(2, n_max + 1):
        ids = _Ids(_windows(stream, 3, None)) if n == 4 else None
        key, cnt = torch.unique(_windows(stream, n, ids), return_counts=True)
        top = torch.sort(cnt, descending=True, stable=True).indices[:count // (n_max - 1)]
        t = torch.full((top.numel(), n_max), -1, dtype=torch.int32, device="cuda")
        t[:, :n] = _fields(key[top], n, ids)
        toks.append(t)
        lens.append(torch.full((top.numel(),), n, dtype=torch.uint8, device="cuda"))
        cnts.append(cnt[top])
    order = torch.sort(torch.cat(cnts), descending=True, stable=True).indices
    return torch.cat(toks)[order], torch.cat(lens)[order]


class _Handle:
    """A library handle, freed before what it borrows."""

    def __init__(self, handle, free, keep=()):
        self.handle, self.free, self.keep = handle, free, keep

    def __del__(self):
        if tfe is not None and getattr(tfe, "lib", None) is not None:
            self.free(self.handle)


def _table(case, seed, toks, lens):
    dim, dtype = case["dim"], DTYPES[case["dtype"]]
    vals = _normal(seed, 2, (lens.numel(), dim), 0.02, dtype)
    t, n, code = toks.cpu().numpy(), lens.cpu().numpy(), tfe.TFE_BF16 if case["dtype"] == "bf16" else tfe.TFE_F32
    stream = torch.cuda.current_stream()
    if case["kind"] == "tiered":
        # Rows in pinned host memory, the most frequent ones cached to begin with.
        host = torch.empty(vals.shape, dtype=dtype, pin_memory=True)
        host.copy_(vals)
        torch.cuda.synchronize()
        desc = tfe.make_desc(t, n, 2, t.shape[1], VOCAB, host, dim, code, 0, hbm_cache_rows=case["cache"],
                             adopt_host_values=1, prefill_rows=case["cache"])
        return _Handle(tfe.tfe_table_load(desc, stream), tfe.tfe_table_free, (host,))
    desc = tfe.make_desc(t, n, 2, t.shape[1], VOCAB, vals, dim, code, 1)
    return _Handle(tfe.tfe_table_load(desc, stream), tfe.tfe_table_free)


def _lookup_inputs(case, seed):
    rows, ctx, S = case["rows"], case.get("ctx", 0), case["steps"]
    calls = case.get("calls", 0)
    if case["kind"] == "tiered" and S == 1:
        # `rows` running sequences: call i sees each one's 3-token window ending at its token i + 2.
        seq = _tokens(seed, 3, rows * (calls + 3)).view(rows, calls + 3)
        tokens = torch.stack([seq[:, i:i + 3] for i in range(calls)]).contiguous()
    else:
        seq, tokens = None, _tokens(seed, 3, max(calls, 1) * rows * (ctx + S)).view(max(calls, 1), rows, ctx + S)
    hidden = _normal(seed, 4, (tokens.shape[0] * rows * S, case["dim"]), 1.0, DTYPES[case["dtype"]])
    return seq, tokens, hidden


def _head_inputs(case, seed):
    return (_normal(seed, 5, (case["vocab"], case["dim"]), 0.1, torch.bfloat16),
            _normal(seed, 6, (case["rows"], case["dim"]), 1.0, torch.bfloat16))


def _ngram_inputs(case, seed):
    tokens = _tokens(seed, 7, case["tokens"])
    if case["doc"]:
        g = _gen(seed, 8)
        ends = torch.randint(0, case["tokens"], (case["tokens"] // case["doc"],), generator=g, device="cuda")
        tokens[ends] = -1  # document separators
    return tokens


def prepare(case, seed):
    kind = case["kind"]
    if kind == "head":
        w, hidden = _head_inputs(case, seed)
        B, K = case["rows"], case["k"]
        head = _Handle(tfe.tfe_head_create(w, case["vocab"], case["dim"], B, K), tfe.tfe_head_free, (w,))
        return {"case": case, "head": head, "hidden": hidden,
                "ids": torch.empty((B, K), dtype=torch.int32, device="cuda"),
                "prob": torch.empty((B, K), dtype=torch.float32, device="cuda")}
    if kind == "ngram":
        return {"case": case, "tokens": _ngram_inputs(case, seed),
                "tuples": torch.zeros((case["top"], case["n"]), dtype=torch.int32, device="cuda"),
                "counts": torch.zeros((case["top"],), dtype=torch.int64, device="cuda")}
    n_max = case.get("n_max", 3)
    toks, lens = _phrases(seed, case["phrases"], n_max)
    seq, tokens, hidden = _lookup_inputs(case, seed)
    T, L = hidden.shape[0], n_max - 1
    state = {"case": case, "table": _table(case, seed, toks, lens), "tokens": tokens, "hidden": hidden,
             "out": torch.empty_like(hidden), "hit": torch.empty(T, dtype=torch.uint8, device="cuda"),
             "slot": torch.empty((T, L) if case.get("multi") else (T,), dtype=torch.int32, device="cuda"),
             "len": torch.empty(T, dtype=torch.uint8, device="cuda")}
    if case.get("candidates"):
        # Predicted next tokens of each sequence: the true one with probability 0.7, at a random place.
        B, K, calls = case["rows"], case["candidates"], case["calls"]
        g = _gen(seed, 9)
        cand = _tokens(seed, 10, calls * B * K).view(calls, B, K)
        put = torch.rand((calls, B), generator=g, device="cuda") < 0.7
        at = torch.randint(0, K, (calls, B, 1), generator=g, device="cuda")
        true = torch.stack([seq[:, i + 3] for i in range(calls)]).unsqueeze(-1)
        cand = torch.where(put.unsqueeze(-1), cand.scatter(2, at, true), cand)
        state["cand"] = cand.contiguous()
        state["tail"] = torch.stack([seq[:, i + 1:i + 3] for i in range(calls)]).contiguous()
        p = torch.rand((calls, B, K), generator=g, device="cuda")
        state["prob"] = (p / p.sum(-1, keepdim=True)).contiguous()
        state["side"] = torch.cuda.Stream()
    return state


# ---- the pass --------------------------------------------------------------------------------


def run(state):
    case = state["case"]
    kind, stream = case["kind"], torch.cuda.current_stream().cuda_stream
    if kind == "head":
        tfe.tfe_head_topk(state["head"].handle, state["hidden"], case["rows"], case["k"], state["ids"], state["prob"],
                          stream)
        return {"ids": state["ids"], "prob": state["prob"]}
    if kind == "ngram":
        written = tfe.tfe_ngram_top(state["tokens"], case["tokens"], VOCAB, case["n"], case["skip"], case["top"],
                                    state["tuples"], state["counts"], stream)
        return {"tuples": state["tuples"], "counts": state["counts"], "written": written}
    table, B, S, ctx = state["table"].handle, case["rows"], case["steps"], case.get("ctx", 0)
    if kind == "tiered":
        ctx = 2 if S == 1 else 0
        T = B * S
        side = state["side"].cuda_stream if "side" in state else None
        for i in range(case["calls"]):
            at = slice(i * T, (i + 1) * T)
            tfe.tfe_lookup_inject(table, state["tokens"][i], B, ctx, S, state["hidden"][at], state["out"][at],
                                  state["hit"][at], state["slot"][at], state["len"][at], tfe.TFE_GATE_SIGMOID, 1.0,
                                  stream)
            if side is not None:
                tfe.tfe_prefetch_scored(table, state["tail"][i], 2, state["cand"][i], state["prob"][i], B,
                                        case["candidates"], case["budget"], side)
        return {"out": state["out"], "hit": state["hit"], "slot": state["slot"], "len": state["len"]}
    gate, scale = (tfe.TFE_GATE_SIGMOID, 1.0) if case["gate"] == "sigmoid" else (tfe.TFE_GATE_CONST, 0.5)
    if case["multi"]:
        tfe.tfe_lookup_inject_multi(table, state["tokens"], B, ctx, S, state["hidden"], state["out"], state["hit"],
                                    state["slot"], tfe.TFE_WEIGHT_LENGTH, gate, scale, stream)
        return {"out": state["out"], "hit": state["hit"], "slot": state["slot"]}
    tfe.tfe_lookup_inject(table, state["tokens"], B, ctx, S, state["hidden"], state["out"], state["hit"], state["slot"],
                          state["len"], gate, scale, stream)
    return {"out": state["out"], "hit": state["hit"], "slot": state["slot"], "len": state["len"]}


# ---- what a pass cannot do without, and what it gives in 64 bits -----------------------------


def work(case):
    kind = case["kind"]
    if kind == "head":
        V, D, B, K = case["vocab"], case["dim"], case["rows"], case["k"]
        return {"bytes": 2 * V * D + 2 * B * D + 8 * B * K, "flops": 2 * B * V * D}
    if kind == "ngram":
        return {"bytes": 4 * case["tokens"] + case["top"] * (4 * case["n"] + 8), "flops": 0}
    T = case["rows"] * case["steps"] * case.get("calls", 1)
    row = case["dim"] * (2 if case["dtype"] == "bf16" else 4)
    values = RETAINED if case.get("multi") else HITS
    # Hidden rows in and out, the matched value rows, one 16-byte index slot a key, results, tokens.
    per = 2 * row + values * row + 16 * (case.get("n_max", 3) - 1) + 6 + 4 * (1 + case.get("ctx", 0))
    return {"bytes": int(T * per), "flops": int(T * values * 8 * case["dim"])}


def tolerance(case):
    kind = case["kind"]
    if kind == "ngram":
        return "exact"
    if kind == "head":
        # float32 sums of bf16 products; neighbours whose logits agree to a rounding may change places.
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    # One rounding to bfloat16 (half an ulp is 2^-9 of the value).
    return {"rel": 4e-3, "max": 1.6e-2}


def exact(case, seed):
    kind = case["kind"]
    if kind == "head":
        w, hidden = _head_inputs(case, seed)
        h = hidden.double()
        logits = torch.cat([h @ w[at:at + 8192].double().t() for at in range(0, case["vocab"], 8192)], 1)
        top = torch.topk(logits, case["k"], dim=1)
        return {"ids": top.indices.to(torch.int32),
                "prob": torch.exp(top.values - torch.logsumexp(logits, 1, keepdim=True))}
    if kind == "ngram":
        tokens, n = _ngram_inputs(case, seed), case["n"]
        ids = _Ids(_windows(tokens, 3, None)) if n == 4 else None
        key, cnt = torch.unique(_windows(tokens, n, ids), return_counts=True)
        key, cnt = key[key >= 0], cnt[key >= 0]
        order = torch.sort(cnt, descending=True, stable=True).indices[case["skip"]:case["skip"] + case["top"]]
        tuples = torch.zeros((case["top"], n), dtype=torch.int32, device="cuda")
        counts = torch.zeros((case["top"],), dtype=torch.int64, device="cuda")
        tuples[:order.numel()] = _fields(key[order], n, ids)
        counts[:order.numel()] = cnt[order]
        return {"tuples": tuples, "counts": counts, "written": int(order.numel())}
    n_max = case.get("n_max", 3)
    toks, lens = _phrases(seed, case["phrases"], n_max)
    vals = _normal(seed, 2, (lens.numel(), case["dim"]), 0.02, DTYPES[case["dtype"]])
    _, tokens, hidden = _lookup_inputs(case, seed)
    S, T = case["steps"], hidden.shape[0]
    flat = tokens.reshape(-1, tokens.shape[-1])
    found = torch.full((T, n_max - 1), -1, dtype=torch.long, device="cuda")  # row of each length's match
    for n in range(2, n_max + 1):
        of = torch.nonzero(lens == n).squeeze(1)
        phr = toks[of, :n]
        ids = _Ids(_windows(phr[:, 1:], 3, None).squeeze(1)) if n == 4 else None
        keys = _windows(phr, n, ids).squeeze(1)
        order = torch.sort(keys).indices
        if flat.shape[1] < n:
            continue
        q = torch.full(flat.shape, -1, dtype=torch.long, device="cuda")
        q[:, n - 1:] = _windows(flat, n, ids)
        q = q[:, -S:].reshape(-1)
        at = torch.searchsorted(keys[order], q).clamp_(max=keys.numel() - 1)
        found[:, n - 2] = torch.where((q >= 0) & (keys[order][at] == q), of[order][at], found[:, n - 2])
    size = torch.arange(2, n_max + 1, device="cuda")
    length = torch.where(found >= 0, size, torch.zeros_like(found))
    if case.get("multi"):
        weight = length.double() / length.sum(1, keepdim=True).clamp(min=1)
    else:
        weight = ((length == length.max(1, keepdim=True).values) & (length > 0)).double()
    out = torch.empty((T, case["dim"]), dtype=torch.float64, device="cuda")
    for at in range(0, T, 4096):
        s = slice(at, at + 4096)
        h = hidden[s].double()
        m = torch.zeros_like(h)
        for j in range(n_max - 1):
            m += weight[s, j:j + 1] * vals[found[s, j].clamp(min=0)].double()
        if case.get("gate", "sigmoid") == "sigmoid":
            rms = [torch.sqrt(x.square().mean(1) + 1e-6) for x in (h, m)]
            g = torch.sigmoid((h * m).sum(1) / (rms[0] * rms[1]) / math.sqrt(case["dim"]))
        else:
            g = torch.full((h.shape[0],), 0.5, dtype=torch.float64, device="cuda")
        out[s] = h + g.unsqueeze(1) * m
    if case.get("multi"):
        mask = ((found >= 0).long() << torch.arange(n_max - 1, device="cuda")).sum(1)
        return {"out": out, "hit": mask.to(torch.uint8), "slot": found.to(torch.int32)}
    best = length.max(1).values
    slot = torch.gather(found, 1, (best - 2).clamp(min=0).unsqueeze(1)).squeeze(1)
    slot = torch.where(best > 0, slot, torch.full_like(slot, -1))
    return {"out": out, "hit": (best > 0).to(torch.uint8), "slot": slot.to(torch.int32), "len": best.to(torch.uint8)}

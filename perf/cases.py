"""The calls whose speed is measured, from the smallest to the largest.

A case is one call (or, for joins and prefixes, the calls that belong
together) of the row-evaluation library on a seeded model and table: the
public entry points lmop_create, lmop_load_weights, lmop_set_prefix(es),
lmop_eval_rows and lmop_release_prefix through their Python binding.
`prepare` makes what a program keeps (a ctx with its weights, the instruction
prefix) and the table; `run` is one pass; `exact` computes the same outputs in
64 bits with plain torch.

Two decoder shapes are used, "8b" (head_dim 128) and "1b" (head_dim 64).  Most
cases run a stack of a few of their layers: a pass through every kernel of the
path, with rounding that has not travelled through a whole model.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_31808_amd import lmop

GROUP = 32

# layers of the whole model, width, query heads, key/value heads, head_dim, MLP width, vocabulary
MODELS = {
    "1b": dict(n_layers=16, d_model=2048, n_heads=32, n_kv_heads=8, head_dim=64, d_ff=8192,
               vocab=128256),
    "8b": dict(n_layers=32, d_model=4096, n_heads=32, n_kv_heads=8, head_dim=128, d_ff=14336,
               vocab=128256),
}
EPS, THETA = 1e-5, 5e5


# ------------------------------------------------------------------ the cases
def _case(name, model, layers, rows, suffix, prefix, answer="enum", choices=24, steps=1,
          weights="int4", head="full", distinct=0, left=0, build="kept", logits=False):
    """rows: table rows; suffix: mean tokens of a row's own text; prefix: tokens of the shared
    instruction; answer: output type, of `choices` options and at most `steps` tokens; distinct:
    number of different texts the rows repeat (0: no repeats); left: left values of a join (rows
    are then right values per left value); build: whether the prefix is kept from before the call
    or computed in it; logits: the call also returns every row's logits."""
    c = dict(name=name, model=model, layers=layers, rows=rows, suffix=suffix, prefix=prefix,
             answer=answer, choices=choices, steps=steps, weights=weights, head=head,
             distinct=distinct, left=left, build=build, logits=logits)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # one question about one value, whole model: what an interactive query waits for
        _case("ask_one_8b", "8b", 32, 1, 60, 512, logits=True),
        # a handful of rows through the small whole model, yes/no, only the two answers' logits:
        # the cheap predicate in front of a cascade
        _case("ask_few_1b", "1b", 16, 5, 33, 384, answer="bool", choices=2, head="restricted"),
        # a small table (or the first rows of a LIMIT query), ragged lengths
        _case("small_table_8b", "8b", 4, 13, 47, 512),
        # numbers read from few rows: nearly all passes are decode steps with a few tokens
        _case("read_numbers_8b", "8b", 4, 9, 44, 256, answer="int", choices=10, steps=8),
        # multi-token options over a medium table: a medium prefill, then medium decode steps
        _case("options_8b", "8b", 4, 61, 60, 512, answer="options", steps=3),
        # integers over a column with many repeated values: deduplication, a large prefill,
        # decode steps of several hundred rows
        _case("map_int_8b", "8b", 4, 1500, 44, 256, answer="int", choices=10, steps=4,
              distinct=420),
        # a join: child prefixes for the left values, then every pair
        _case("join_8b", "8b", 4, 24, 20, 320, answer="bool", choices=2, left=23),
        # one long prompt over a whole data subset, answer of up to 3 tokens
        _case("long_prompt_8b", "8b", 4, 1, 6200, 256, answer="options", steps=3),
        # a new instruction: its prefix is computed and the answer read from its end
        _case("new_prefix_8b", "8b", 4, 1, 0, 1000, build="call", logits=True),
        # the filter over a table, the main workload: full batches
        _case("filter_8b", "8b", 4, 550, 60, 512),
        # the same over FP8 weights
        _case("filter_fp8_8b", "8b", 4, 150, 60, 512, weights="fp8"),
        # the whole small model over a table, yes/no
        _case("filter_1b", "1b", 16, 1000, 40, 384, answer="bool", choices=2),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ones' ranges: any kind of call, at any size up to the largest."""
    model = rng.choice(["8b", "8b", "8b", "1b"])
    layers = rng.randint(3, 5) if model == "8b" else rng.randint(6, 16)
    prefix = _log_uniform(rng, 128, 1024)
    weights = rng.choice(["int4", "int4", "int4", "fp8"])
    head = rng.choice(["full", "full", "full", "restricted"])
    kind = rng.choice(["filter", "filter", "small", "int", "options", "join", "long", "prefix"])
    budget = 26000  # suffix tokens
    if kind == "filter":
        suffix = _log_uniform(rng, 24, 90)
        rows = _log_uniform(rng, 60, budget // suffix)
        ans = rng.choice([("bool", 2), ("enum", rng.randint(3, 40))])
        return _case(None, model, layers, rows, suffix, prefix, ans[0], ans[1], 1, weights, head)
    if kind == "small":
        ans = rng.choice([("bool", 2), ("enum", rng.randint(3, 40))])
        return _case(None, model, layers, _log_uniform(rng, 1, 40), _log_uniform(rng, 16, 90),
                     prefix, ans[0], ans[1], 1, weights, head)
    if kind == "int":
        rows = _log_uniform(rng, 2, 1500)
        distinct = 0 if rows < 100 else _log_uniform(rng, 60, min(rows, 450))
        return _case(None, model, layers, rows, _log_uniform(rng, 24, 56), prefix, "int", 10,
                     rng.randint(2, 8 if rows < 100 else 4), weights, head, distinct)
    if kind == "options":
        return _case(None, model, layers, _log_uniform(rng, 2, 300), _log_uniform(rng, 24, 80),
                     prefix, "options", rng.randint(8, 32), rng.randint(2, 3), weights, head)
    if kind == "join":
        left = _log_uniform(rng, 4, 30)
        return _case(None, model, layers, _log_uniform(rng, 4, 30), rng.randint(10, 24), prefix,
                     "bool", 2, 1, weights, head, 0, left)
    if kind == "long":
        return _case(None, model, layers, 1, _log_uniform(rng, 600, 7000), min(prefix, 512),
                     "options", rng.randint(8, 32), rng.randint(1, 3), weights, head)
    return _case(None, model, layers, 1, 0, _log_uniform(rng, 100, 2000), "enum", 24, 1, weights,
                 "full", 0, 0, "call", True)


# ------------------------------------------------------------------ model and table
def _shape(case):
    m = dict(MODELS[case["model"]])
    m["n_layers"] = case["layers"]
    return SimpleNamespace(group_size=GROUP, rms_eps=EPS, rope_theta=THETA, **m)


def _quantise_int4(w):
    """Symmetric int4, one fp16 scale per 32 input features; two codes a byte, the even feature
    in the low half."""
    n, k = w.shape
    g = w.view(n, k // GROUP, GROUP)
    s = (g.abs().amax(-1) / 7.0).to(torch.float16)
    q = torch.round(g / s.float().unsqueeze(-1)).clamp_(-8, 7).to(torch.int8).view(n, k)
    return ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous(), s.contiguous()


def _quantise_fp8(w):
    """E4M3 codes with one fp32 scale per output row."""
    s = w.abs().amax(-1) / 448.0
    q = (w / s.unsqueeze(-1)).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.view(torch.uint8).contiguous(), s.contiguous()


def _weights(case, seed, device):
    """Random weights N(0, 0.02), quantised; norm gains spread around 1."""
    sh = _shape(case)
    gen = torch.Generator(device=device)
    gen.manual_seed(seed * 7919 + 17)
    fmt = "fp8_e4m3" if case["weights"] == "fp8" else "int4_g32"

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=device, dtype=torch.float32).mul_(0.02)

    def mat(n, k):
        q, s = (_quantise_fp8 if fmt == "fp8_e4m3" else _quantise_int4)(normal(n, k))
        return SimpleNamespace(qweight=q, scales=s, n=n, k=k, fmt=fmt)

    def gain():
        return 1.0 + 5.0 * normal(sh.d_model)

    nq, nkv = sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    emb = normal(sh.vocab, sh.d_model).to(torch.float16)
    head = normal(sh.vocab, sh.d_model).to(torch.float16)
    layers = [SimpleNamespace(
        attn_norm=gain(), mlp_norm=gain(), wq=mat(nq, sh.d_model), wk=mat(nkv, sh.d_model),
        wv=mat(nkv, sh.d_model), wo=mat(sh.d_model, nq), w_gate=mat(sh.d_ff, sh.d_model),
        w_up=mat(sh.d_ff, sh.d_model), w_down=mat(sh.d_model, sh.d_ff))
        for _ in range(sh.n_layers)]
    return SimpleNamespace(tok_embedding=emb, lm_head=head, final_norm=gain(), layers=layers)


def _trie(options):
    """Token strings as an automaton: a state per distinct beginning, ends accepting."""
    children, ends = [{}], []
    for o in options:
        st = 0
        for t in o:
            if t not in children[st]:
                children[st][t] = len(children)
                children.append({})
            st = children[st][t]
        ends.append(st)
    off, tok, nxt = [0], [], []
    for c in children:
        tok += list(c.keys())
        nxt += list(c.values())
        off.append(len(tok))
    acc = np.zeros(len(children), dtype=np.uint8)
    acc[ends] = 1
    return SimpleNamespace(n_states=len(children), edge_offset=np.array(off, np.int32),
                           edge_token=np.array(tok, np.int32), edge_next=np.array(nxt, np.int32),
                           accepting=acc)


def _lengths(rng, case, n):
    mean = case["suffix"]
    if mean == 0:
        return np.zeros(n, dtype=np.int64)
    if n == 1:
        return np.array([mean], dtype=np.int64)
    if case["answer"] == "int" or case["left"]:
        return rng.integers(max(1, mean * 6 // 10), mean * 14 // 10 + 1, size=n)
    mu = math.log(mean) - 0.75 * 0.75 / 2.0
    return np.clip(np.rint(rng.lognormal(mu, 0.75, size=n)), 4, 512).astype(np.int64)


def _table(case, seed):
    """Prefix tokens, left values, row texts (with their left value) and output type."""
    rng = np.random.default_rng([seed, 5])
    V = MODELS[case["model"]]["vocab"]

    def text(n):
        return rng.integers(0, V, size=int(n)).astype(np.int32)

    prefix = text(case["prefix"])
    left = [text(n) for n in _lengths(rng, case, case["left"])] if case["left"] else []
    texts = [text(n) for n in _lengths(rng, case, case["distinct"] or case["rows"])]
    row_left = None
    if left:  # every pair, left-major
        row_left = np.repeat(np.arange(len(left)), len(texts))
        rows = [t for _ in left for t in texts]
    elif case["distinct"]:  # repeated values, the common ones far more often
        p = np.arange(1, len(texts) + 1, dtype=np.float64) ** -1.1
        rows = [texts[i] for i in rng.choice(len(texts), size=case["rows"], p=p / p.sum())]
    else:
        rows = texts
    ids = [int(t) for t in rng.choice(V, size=case["choices"] * 3 + 9, replace=False)]
    eos, allowed, options = -1, None, None
    if case["answer"] == "options":  # 8 first tokens shared by all options
        heads, rest = ids[:8], ids[8:-1]
        options = []
        for i in range(case["choices"]):
            n = 1 if i < 2 else int(rng.integers(2, case["steps"] + 1)) if case["steps"] > 1 else 1
            first = heads[i] if n == 1 and i < 8 else heads[2 + i % 6]
            o = tuple([first] + [rest[(2 * i + j) % len(rest)] for j in range(n - 1)])
            if o not in options:
                options.append(o)
        allowed = _trie(options)
    else:
        allowed = np.array(ids[:case["choices"]], dtype=np.int32)
        eos = ids[-1] if case["answer"] == "int" else -1
    lens = np.array([len(r) for r in rows], dtype=np.int64)
    offsets = np.zeros(len(rows) + 1, dtype=np.int64)
    np.cumsum(lens, out=offsets[1:])
    tokens = np.concatenate(rows).astype(np.int32) if offsets[-1] else np.zeros(0, np.int32)
    return SimpleNamespace(prefix=prefix, left=left, rows=rows, row_left=row_left, tokens=tokens,
                           offsets=offsets, allowed=allowed, eos=eos)


KINDS = {"bool": lmop.LMOP_BOOL, "enum": lmop.LMOP_ENUM, "int": lmop.LMOP_INT,
         "options": lmop.LMOP_AUTOMATON}


def prepare(case, seed):
    """A ctx with its weights, the instruction's prefix (unless the call computes it), the table."""
    table = _table(case, seed)
    longest = max(len(r) for r in table.rows) + max([len(t) for t in table.left], default=0)
    ctx = lmop.Context(_shape(case), device=0,
                       max_seq=max(2048, len(table.prefix) + longest + case["steps"] + 1))
    ctx.load_weights(_weights(case, seed, "cuda"))
    torch.cuda.synchronize()
    prefix = ctx.set_prefix(table.prefix) if case["build"] == "kept" else None
    return SimpleNamespace(case=case, ctx=ctx, table=table, prefix=prefix)


def run(state):
    case, t, ctx = state.case, state.table, state.ctx
    prefix, row_prefix, children = state.prefix, None, []
    if case["build"] == "call":
        prefix = ctx.set_prefix(t.prefix)
    if t.left:
        children = ctx.set_prefixes(t.left, parent=prefix)
        row_prefix = [children[i] for i in t.row_left]
    out, logits = ctx.eval_rows(t.tokens, t.offsets, KINDS[case["answer"]], t.allowed, eos=t.eos,
                                max_tokens=case["steps"], prefix=prefix, row_prefix=row_prefix,
                                head_restricted=case["head"] == "restricted",
                                debug_logits=case["logits"])
    for p in children:
        ctx.release_prefix(p)
    if case["build"] == "call":
        ctx.release_prefix(prefix)
    got = {"logprob": out["logprob"], "logprob_full": out["logprob_full"]}
    if case["logits"]:
        got["logits"] = logits
    if len(t.rows) >= 200:
        # the answers themselves: in a small table one near-tie that rounds the other way
        # would be more than the share of ties that a comparison can allow
        got["value"], got["tokens"] = out["value"], out["tokens"]
    return got


# ------------------------------------------------------------------ what a pass cannot do without
def _distinct_rows(case):
    """Rows evaluated (a column of repeated values: about how many different ones are drawn)."""
    if case["left"]:
        return case["rows"] * case["left"]
    if case["distinct"]:
        p = np.arange(1, case["distinct"] + 1, dtype=np.float64) ** -1.1
        return int(round(float(np.sum(1.0 - (1.0 - p / p.sum()) ** case["rows"]))))
    return case["rows"]


def work(case):
    m = MODELS[case["model"]]
    d, hd, F, V, L = m["d_model"], m["head_dim"], m["d_ff"], m["vocab"], case["layers"]
    nq, nkv = m["n_heads"] * hd, m["n_kv_heads"] * hd
    kv_par = 2 * nkv * d                       # k and v: for every token in every layer
    rest_par = 2 * nq * d + 3 * d * F          # q, o, MLP: in the last layer for last tokens only
    rows = _distinct_rows(case)
    # (sequences, tokens each, keys before them, tokens whose answer is wanted) of the first pass
    runs = [(rows, case["suffix"], case["prefix"] + (case["suffix"] if case["left"] else 0))]
    if case["left"]:
        runs.append((case["left"], case["suffix"], case["prefix"]))
    if case["build"] == "call":
        runs = [(1, case["prefix"], 0)]
    flops = kv_rw = tokens = 0.0
    for n, t, before in runs:
        tokens += n * t
        flops += 2.0 * n * t * (L * kv_par + (L - 1) * rest_par) + 2.0 * n * rest_par
        flops += 4.0 * nq * n * ((L - 1) * (t * before + t * (t + 1) / 2.0) + before + t)
        kv_rw += 4.0 * nkv * L * (n * t)       # written keys and values, fp16
    kv_rw += 4.0 * nkv * L * (0 if case["build"] == "call" else case["prefix"])
    n_head = case["choices"] if case["head"] == "restricted" else V
    passes = 1
    # further steps: one token per row still open.  Of ten digits and the end every eleventh
    # choice ends a number; two of the options' eight first tokens are whole options, and half
    # of the longer options end with their second token
    open_ = rows if case["answer"] == "int" else rows * 0.75
    for _ in range(case["steps"] - 1):
        passes += 1
        flops += open_ * (2.0 * L * (kv_par + rest_par) + 2.0 * n_head * d +
                          4.0 * nq * L * (case["prefix"] + case["suffix"]))
        kv_rw += 4.0 * nkv * L * (case["prefix"] + open_ * case["suffix"])
        open_ *= 10.0 / 11.0 if case["answer"] == "int" else 0.5
    flops += 2.0 * rows * n_head * d
    per_weight = 1.0 if case["weights"] == "fp8" else 0.5625
    weights = (kv_par + rest_par) * L * per_weight + 2.0 * n_head * d
    bytes_ = passes * weights + kv_rw + 2.0 * d * tokens + 56.0 * rows
    if case["logits"]:
        bytes_ += 4.0 * case["rows"] * V
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # fp16 operands, fp32 sums.  Against 64 bits the log-probabilities (differences of logits)
    # of a stack of 4 layers are up to 0.0033 off, those and the logits of a whole model 0.007;
    # another implementation's rounding is as far off the other way, and seeds differ
    if case["steps"] > 1:
        # a near-tie that rounds the other way changes the row's further steps
        return {"rel": 2e-2, "max": 0.5, "differ": 1e-2}
    if case["layers"] > 5:
        return {"rel": 2.5e-2, "max": 0.15, "differ": 1e-2}
    return {"rel": 1e-2, "max": 0.05, "differ": 1e-2}


# ------------------------------------------------------------------ the same in 64 bits
def _dequantise(m):
    if m.fmt == "fp8_e4m3":
        return m.qweight.view(torch.float8_e4m3fn).double() * m.scales.double().unsqueeze(-1)
    b = m.qweight.to(torch.int16)
    q = torch.stack([b & 15, b >> 4], dim=-1).view(m.n, m.k)
    q = torch.where(q > 7, q - 16, q).double()
    return (q.view(m.n, m.k // GROUP, GROUP) * m.scales.double().unsqueeze(-1)).view(m.n, m.k)


def _rms_norm(x, gain):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()


def _rotate(x, pos):
    half = x.shape[-1] // 2
    inv = THETA ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    a = pos.double()[:, None] * inv[None, :]
    c, s = a.cos()[:, None, :], a.sin()[:, None, :]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x1 * s + x2 * c], dim=-1)


class _Sequences:
    """Token sequences that each continue a shared prefix, run layer by layer; keys and values
    are kept, so that sequences can grow by one token."""

    def __init__(self, case, w, prefix, seqs, device):
        self.sh, self.w, self.dev = _shape(case), w, device
        self.P = len(prefix)
        self.seqs = [list(map(int, s)) for s in seqs]
        toks = np.concatenate([np.asarray(prefix, np.int64)] +
                              [np.asarray(s, np.int64) for s in self.seqs])
        pos = np.concatenate([np.arange(self.P)] + [self.P + np.arange(len(s)) for s in self.seqs])
        starts = np.cumsum([self.P] + [len(s) for s in self.seqs])
        # where in the flat arrays each sequence's tokens are
        self.at = [list(range(starts[i], starts[i + 1])) for i in range(len(self.seqs))]
        self.k, self.v = [None] * self.sh.n_layers, [None] * self.sh.n_layers
        groups = [(None, 0, self.P)] if self.P else []
        groups += [(i, 0, len(s)) for i, s in enumerate(self.seqs) if s]
        x = self._layers(toks, pos, groups, 0)
        last = [self.at[i][-1] if s else self.P - 1 for i, s in enumerate(self.seqs)]
        self.hidden = x[torch.tensor(last, device=device)]

    def grow(self, rows, tokens):
        """Appends one token to each of `rows`; self.hidden becomes theirs, in that order."""
        base = self.k[0].shape[0] if self.k else 0
        pos, groups = [], []
        for j, (i, t) in enumerate(zip(rows, tokens)):
            pos.append(self.P + len(self.seqs[i]))
            self.seqs[i].append(int(t))
            self.at[i].append(base + j)
            groups.append((i, len(self.seqs[i]) - 1, len(self.seqs[i])))
        self.hidden = self._layers(np.asarray(tokens, np.int64), np.asarray(pos), groups, base)

    def _layers(self, toks, pos, groups, base):
        sh, dev = self.sh, self.dev
        T = len(toks)
        x = self.w.tok_embedding[torch.as_tensor(toks, device=dev)].double()
        pos = torch.as_tensor(pos, device=dev)
        pieces = []  # at most 1,024 queries of one sequence
        for i, a, b in groups:
            pieces += [(i, q, min(q + 1024, b)) for q in range(a, b, 1024)]
        pieces.sort(key=lambda g: g[2] - g[1])
        for l, L in enumerate(self.w.layers):
            h = _rms_norm(x, L.attn_norm)
            q = _rotate((h @ _dequantise(L.wq).T).view(T, sh.n_heads, sh.head_dim), pos)
            k = _rotate((h @ _dequantise(L.wk).T).view(T, sh.n_kv_heads, sh.head_dim), pos)
            v = (h @ _dequantise(L.wv).T).view(T, sh.n_kv_heads, sh.head_dim)
            self.k[l] = k if base == 0 else torch.cat([self.k[l], k])
            self.v[l] = v if base == 0 else torch.cat([self.v[l], v])
            o = torch.empty_like(q)
            at = 0
            while at < len(pieces):  # pieces of about the same length together
                n = 1
                while at + n < len(pieces):
                    i, a, b = pieces[at + n]
                    keys = self.P + len(self.seqs[i] if i is not None else ())
                    if (n + 1) * (b - a) * max(keys, 1) > 2_000_000:
                        break
                    n += 1
                self._attend(q, o, l, pieces[at:at + n], base)
                at += n
            x = x + o.view(T, -1) @ _dequantise(L.wo).T
            h = _rms_norm(x, L.mlp_norm)
            act = torch.nn.functional.silu(h @ _dequantise(L.w_gate).T)
            x = x + (act * (h @ _dequantise(L.w_up).T)) @ _dequantise(L.w_down).T
        return x

    def _attend(self, q, o, l, pieces, base):
        sh, dev = self.sh, self.dev
        G, hd = sh.n_heads // sh.n_kv_heads, sh.head_dim
        Lq = max(b - a for _, a, b in pieces)
        where, keys, see = [], [], []
        for i, a, b in pieces:
            own = list(range(self.P)) if i is None else self.at[i]
            where.append([own[min(j, b - 1)] - base for j in range(a, a + Lq)])
            keys.append((list(range(self.P)) if i is not None else []) + own[:b])
            before = self.P if i is not None else 0
            see.append([before + min(j, b - 1) + 1 for j in range(a, a + Lq)])
        Lk = max(len(s) for s in keys)
        keys = torch.tensor([s + [s[0]] * (Lk - len(s)) for s in keys], device=dev)
        see = torch.tensor(see, device=dev)
        where = torch.tensor(where, device=dev)
        n = len(pieces)
        kk = self.k[l][keys].permute(0, 2, 3, 1).contiguous()            # n, kv head, hd, key
        vv = self.v[l][keys].permute(0, 2, 1, 3).contiguous()            # n, kv head, key, hd
        qq = q[where].view(n, Lq, sh.n_kv_heads, G, hd).permute(0, 2, 1, 3, 4)
        qq = qq.reshape(n, sh.n_kv_heads, Lq * G, hd)
        s = (qq @ kk) / math.sqrt(hd)
        ok = torch.arange(Lk, device=dev)[None, None, :] < see[:, :, None]
        ok = ok.repeat_interleave(G, dim=1)[:, None]
        p = torch.softmax(s.masked_fill(~ok, -math.inf), dim=-1)
        got = (p @ vv).view(n, sh.n_kv_heads, Lq, G, hd).permute(0, 2, 1, 3, 4)
        o[where.reshape(-1)] = got.reshape(n * Lq, sh.n_heads, hd)


def exact(case, seed, device="cuda"):
    t = _table(case, seed)
    w = _weights(case, seed, device)
    place, first, seqs = {}, [], []
    for r, text in enumerate(t.rows):
        own = np.concatenate([t.left[t.row_left[r]], text]) if t.left else text
        key = own.tobytes()
        if key not in place:
            place[key] = len(seqs)
            seqs.append(own)
        first.append(place[key])
    S = _Sequences(case, w, t.prefix, seqs, device)
    n = len(seqs)
    value, lp, lpf = np.zeros(n, np.int64), np.zeros(n), np.zeros(n)
    tokens = np.full((n, 8), -1, np.int32)
    aut = t.allowed if case["answer"] == "options" else None
    state, live, logits = np.zeros(n, np.int64), list(range(n)), None
    for step in range(case["steps"]):
        if step:
            S.grow(live, [tokens[i, step - 1] for i in live])
        hidden = _rms_norm(S.hidden, w.final_norm)
        z_all = [hidden[a:a + 256] @ w.lm_head.double().T for a in range(0, len(live), 256)]
        if case["logits"]:
            logits = torch.cat(z_all)[first][:, None].cpu().numpy()
        nxt = []
        for j, i in enumerate(live):
            z = z_all[j // 256][j % 256]
            if aut is not None:
                e = range(aut.edge_offset[state[i]], aut.edge_offset[state[i] + 1])
                choice = [int(aut.edge_token[x]) for x in e]
            else:
                choice = [int(x) for x in t.allowed]
                if case["answer"] == "int" and step:
                    choice.append(t.eos)
            za = z[torch.tensor(choice, device=device)]
            b = int(torch.argmax(za))
            lp[i] += float(za[b] - torch.logsumexp(za, 0))
            lpf[i] += float(za[b] - torch.logsumexp(z, 0))
            tokens[i, step] = choice[b]
            if aut is not None:
                state[i] = aut.edge_next[aut.edge_offset[state[i]] + b]
                done = aut.edge_offset[state[i]] == aut.edge_offset[state[i] + 1]
                value[i] = state[i] if done else -1
            elif case["answer"] == "int":
                done = choice[b] == t.eos
                value[i] = value[i] if done else value[i] * 10 + b
            else:
                value[i], done = b, True
            if not done:
                nxt.append(i)
        live = nxt
        if not live:
            break
    got = {"logprob": lp[first], "logprob_full": lpf[first]}
    if case["head"] == "restricted":
        got["logprob_full"] = np.full(len(first), np.nan)
    if case["logits"]:
        got["logits"] = logits
    if len(t.rows) >= 200:
        got["value"], got["tokens"] = value[first], tokens[first]
    return got

"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values.  Five kinds of work cover the entry points of
the library:

* `decode`: a serving episode.  The contexts of a batch are taken in
  (sd_index_build of the requests), first drafts are made, and `steps` decode
  steps follow: acceptance against the target model's tokens, append, next drafts.
  `calls` says how the program makes a step: "fused" (one
  sd_accept_append_speculate), "two" (sd_accept_append, sd_speculate) or
  "separate" (sd_accept, sd_index_append, sd_speculate).  With `graph` the
  episode is a captured HIP graph that is replayed, as in a serving loop with
  static buffers; otherwise every call is made from the host.
* `draft`: sd_speculate alone, for contexts that are already in their slots.
* `build`: a server starts: the index over earlier outputs is built, and the
  waiting requests get their first drafts from it.
* `insert`: a server that keeps its index up to date: the index over earlier
  outputs is built, then several batches of finished outputs are inserted, the
  in-flight requests drafting anew after each.
* `entropy`: the predictor of how well drafting will work on a corpus.

Token streams are synthetic, of the two processes and the parameters of the
benchmark configurations: documents and contexts pasted together from spans of a
pool of templates with some tokens mutated (agentic traces), or independent
tokens of a Zipf law (open-ended text).  The target model says what the
unmutated template says next.  What it says about each step's drafts, and the
tokens that a step with separate calls appends, are recorded once in `prepare`:
they stand for the output of the target model, which is not part of the library.
"""
import math

import numpy as np
import torch

import paper_2411_04975_amd as sd

# (depth bound D, longest pattern P, alpha, min_score) of the benchmark configurations
LIMITS = ((24, 16, 1.0, 0.1), (64, 32, 1.0, 0.1), (64, 32, 2.0, 0.05), (32, 16, 1.0, 0.1))
VOCABS = (32000, 128256, 152064)

BASE = dict(kind="decode", process="templated", vocab=128256, mut=0.05, templates=200,
            corpus=2_200_000, batch=64, ctx=8192, ragged=False, slots=False, D=64, P=32,
            alpha=1.0, min_score=0.1, linear=0, den_mode=0, tau=0.0, steps=8, calls="fused",
            graph=False, rounds=0, new_docs=0, new_len=0)


def _case(name, **over):
    c = dict(BASE, **over)
    c["name"] = name
    return c


def listed():
    zipf = dict(process="zipf", vocab=152064, corpus=10_000_000, batch=256, ctx=4096, D=32, P=16)
    large = dict(mut=0.03, templates=5000, corpus=10_000_000, batch=256, ctx=16384, alpha=2.0,
                 min_score=0.05)
    streaming = dict(templates=10000, corpus=100_000_000, batch=512)
    return [
        # one user at a prompt: a single request drafts; the latency of the smallest call
        _case("draft_one", kind="draft", batch=1, ctx=3001),
        # an agent server at moderate load, its loop driven from the host, one call per step
        _case("decode_agentic"),
        # the headline configuration: long contexts, large trees, the loop captured in a graph
        _case("decode_large", graph=True, **large),
        # open-ended chat: little repetition, frequent last tokens, wide first-token buckets
        _case("decode_lowrep", graph=True, **zipf),
        # the largest index and a batch of two requests per compute unit
        _case("decode_streaming", graph=True, steps=16, **streaming),
        # chain drafts behind a hybrid gate, a program that makes every call of a step by itself,
        # requests of unequal length spread over the slots
        _case("decode_ragged_chain", process="templated", corpus=1_234_567, batch=37, ctx=2999,
              ragged=True, slots=True, linear=1, den_mode=1, tau=2.0, calls="separate"),
        # drafting as throughput work: many more requests than compute units
        _case("draft_8192", kind="draft", **dict(large, batch=8192)),
        # server start on the headline corpus, on low-repetition text, and on the largest corpus
        _case("build_large", kind="build", **large),
        _case("build_lowrep", kind="build", **zipf),
        _case("build_streaming", kind="build", **streaming),
        # an agent server that adds the outputs of finished requests to its index
        _case("insert_agentic", kind="insert", rounds=4, new_docs=64, new_len=500),
        # is this corpus worth drafting from?
        _case("entropy_large", kind="entropy", **dict(large, batch=0, ctx=0)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("decode", "draft", "build", "insert", "entropy"), (9, 4, 3, 2, 1))[0]
    process = rng.choices(("templated", "zipf"), (2, 1))[0]
    D, P, alpha, min_score = rng.choice(LIMITS)
    corpus = {"decode": (20_000, 20_000_000), "draft": (20_000, 20_000_000),
              "build": (20_000, 40_000_000), "insert": (100_000, 10_000_000),
              "entropy": (20_000, 20_000_000)}[kind]
    c = dict(BASE, kind=kind, process=process, vocab=rng.choice(VOCABS),
             mut=rng.choice((0.03, 0.05)), corpus=_log_int(rng, *corpus), D=D, P=P, alpha=alpha,
             min_score=min_score, ragged=rng.random() < 0.4, slots=rng.random() < 0.3,
             calls=rng.choice(("fused", "fused", "two", "separate")), graph=rng.random() < 0.5)
    c["templates"] = max(10, min(10000, c["corpus"] // rng.randint(2000, 10000)))
    if rng.random() < 0.15:
        c["linear"], c["tau"] = 1, 2.0
    if rng.random() < 0.15:
        c["den_mode"] = 1
    if kind == "draft":
        c["batch"] = _log_int(rng, 1, 8192)
        c["ctx"] = min(_log_int(rng, 128, 16384), (1 << 26) // c["batch"])
    elif kind == "entropy":
        c["batch"] = c["ctx"] = 0
    else:
        c["batch"] = _log_int(rng, 1, 512)
        c["ctx"] = min(_log_int(rng, 128, 16384), (1 << 22) // c["batch"])
    if kind == "insert":
        c["rounds"], c["new_docs"] = rng.randint(1, 6), _log_int(rng, 1, 256)
        c["new_len"] = _log_int(rng, 32, 1000)
    return c


# ---- token streams, made on the GPU ----------------------------------------------------------


class _Streams:
    """Documents and contexts of one process, drawn from one seed."""

    def __init__(self, case, seed):
        self.case, self.dev = case, torch.device("cuda", 0)
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(0x5D0000000 + int(seed))
        if case["process"] == "templated":
            self.span, self.t_len = (16, 256), 1024
            self.pool = self._ints(0, case["vocab"], case["templates"] * self.t_len)
        else:
            w = 1.0 / torch.arange(1, case["vocab"] + 1, dtype=torch.float64, device=self.dev) ** 1.1
            self.cdf = torch.cumsum(w, 0)
            self.cdf /= self.cdf[-1].clone()

    def _ints(self, lo, hi, n, dtype=torch.int32):
        return torch.randint(lo, hi, (n,), generator=self.g, device=self.dev, dtype=dtype)

    def _zipf(self, n):
        out = torch.empty(n, dtype=torch.int32, device=self.dev)
        for a in range(0, n, 1 << 24):
            u = torch.rand(min(n - a, 1 << 24), generator=self.g, device=self.dev, dtype=torch.float64)
            out[a:a + u.numel()] = torch.searchsorted(self.cdf, u).clamp_(max=self.case["vocab"] - 1)
        return out

    def _offsets(self, lens):
        off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=self.dev)
        torch.cumsum(lens, 0, out=off[1:])
        return off

    def corpus(self, total):
        """Documents of 200 to 2000 tokens (2000 for the Zipf process), `total` tokens together."""
        if self.case["process"] == "zipf":
            lens = torch.full((-(-total // 2000),), 2000, dtype=torch.int64, device=self.dev)
        else:
            lens = self._ints(200, 2001, total // 200 + 1, torch.int64)
        ends = torch.cumsum(lens, 0)
        n = int((ends < total).sum()) + 1
        lens = lens[:n].clone()
        lens[-1] -= ends[n - 1] - total
        return self.sequences(lens, total)

    def sequences(self, lens, total):
        """(tokens, offsets) of sequences of the given lengths; remembers where the last span of
        each sequence would go on."""
        off = self._offsets(lens)
        if self.case["process"] == "zipf":
            return self._zipf(total), off
        # spans one after the other over the whole stream; a span is cut at its sequence's end,
        # and the position within the template restarts with the next one
        lo, hi = self.span
        n_spans = total // ((lo + hi) // 2) + total // (4 * hi) + 64
        sizes = self._ints(lo, hi + 1, n_spans, torch.int64)
        ends = torch.cumsum(sizes, 0)
        sizes, ends = sizes[ends - sizes < total], ends[ends - sizes < total]
        # sequences start spans of their own: the cuts are span ends as well
        ends = torch.unique(torch.cat((ends[ends < total], off[1:])))
        starts = torch.cat((ends.new_zeros(1), ends[:-1]))
        n = ends.numel()
        where = (torch.rand(n, generator=self.g, device=self.dev, dtype=torch.float64)
                 * (self.t_len - (ends - starts) + 1)).long().clamp_(min=0)
        base = self._ints(0, self.case["templates"], n, torch.int64) * self.t_len
        first = torch.repeat_interleave(base + where - starts, ends - starts, output_size=total)
        tokens = self.pool[first.add_(torch.arange(total, device=self.dev))]
        del first
        change = torch.rand(total, generator=self.g, device=self.dev) < self.case["mut"]
        tokens = torch.where(change, self._ints(0, self.case["vocab"], total), tokens)
        last = torch.searchsorted(ends, off[1:])
        self.next_base, self.next_at = base[last], where[last] + (ends - starts)[last]
        return tokens, off

    def contexts(self):
        """(tokens, offsets, slot ids or None, lengths' sum) of the case's requests."""
        c = self.case
        B = c["batch"]
        if c["ragged"]:
            lens = self._ints(max(1, c["ctx"] // 4), c["ctx"] + 1, B, torch.int64)
        else:
            lens = torch.full((B,), c["ctx"], dtype=torch.int64, device=self.dev)
        total = int(lens.sum())
        tokens, off = self.sequences(lens, total)
        slots = None
        if c["slots"]:
            slots = torch.randperm(B, generator=self.g, device=self.dev).to(torch.int32)
        return tokens, off, slots, total

    def futures(self, n):
        """What the target model says after each context, int32[batch, n]."""
        if self.case["process"] == "zipf":
            return self._zipf(self.case["batch"] * n).reshape(-1, n)
        at = (self.next_at[:, None] + torch.arange(n, device=self.dev)) % self.t_len
        return self.pool[self.next_base[:, None] + at]


# ---- what a program has in hand before the call ----------------------------------------------


class _State:
    """The handle and buffers of one program; the handle goes with it."""

    def __init__(self, case, capacity, batch):
        self.case, self.dev, self.ctx = case, torch.device("cuda", 0), None
        nodes = int(math.floor(case["alpha"] * case["P"]))
        longest = max(1, case["ctx"]) + (case["steps"] + 1) * (nodes + 1)
        self.ctx = sd.sd_create(case["vocab"], case["D"], case["P"], case["alpha"],
                                case["min_score"], max(1, batch), longest, capacity, 0,
                                den_mode=case["den_mode"], linear=case["linear"], tau=case["tau"])
        self.nodes, self.graph = nodes, None

    def __del__(self):
        if self.ctx is not None:
            self.graph = None
            sd.sd_destroy(self.ctx)
            self.ctx = None

    def trees(self):
        return sd.Trees(self.case["batch"], self.nodes, self.dev)

    def build_global(self):
        sd.sd_index_build(self.ctx, sd.SD_SCOPE_GLOBAL, None, self.docs, self.doc_off,
                          self.case["corpus"])

    def take_requests(self):
        sd.sd_index_build(self.ctx, sd.SD_SCOPE_REQUESTS, self.slots, self.requests,
                          self.request_off, self.request_tokens)


def _depths(parents):
    """Depth of every draft node (children of the matched node: 1), int64[batch, nodes]."""
    up = parents.long()
    depth = torch.ones_like(up)
    hops = 1
    while hops < parents.shape[1]:
        at = up.clamp(min=0)
        more = up >= 0
        depth = depth + torch.where(more, depth.gather(1, at), torch.zeros_like(depth))
        up = torch.where(more, up.gather(1, at), up)
        hops *= 2
    return depth


def _record(s, streams):
    """Plays the episode once and keeps what the target model says to every step's drafts."""
    B, T, mn, i32 = s.case["batch"], s.case["steps"], s.nodes, torch.int32
    future = streams.futures((T + 1) * (mn + 1) + 1)
    pos = torch.zeros((B, 1), dtype=torch.int64, device=s.dev)
    s.targets = torch.zeros((T, B, mn + 1), dtype=i32, device=s.dev)
    s.accept_len = torch.zeros((T, B), dtype=i32, device=s.dev)
    s.accept_path = torch.full((T, B, mn), -1, dtype=i32, device=s.dev)
    s.bonus = torch.zeros((T, B), dtype=i32, device=s.dev)
    s.appended = []
    s.take_requests()
    sd.sd_speculate(s.ctx, s.slots, s.out)
    for t in range(T):
        s.targets[t, :, :1] = future.gather(1, pos)
        s.targets[t, :, 1:] = future.gather(1, pos + _depths(s.out.parents))
        sd.sd_accept(s.ctx, s.out, B, s.targets[t], s.accept_len[t], s.accept_path[t], s.bonus[t])
        n = s.accept_len[t].long()[:, None]
        taken = s.out.tokens.gather(1, s.accept_path[t].long().clamp(min=0))
        row = torch.cat((taken, torch.zeros((B, 1), dtype=i32, device=s.dev)), 1)
        row.scatter_(1, n, s.bonus[t][:, None])
        new = row[torch.arange(mn + 1, device=s.dev) <= n].contiguous()
        new_off = torch.zeros(B + 1, dtype=i32, device=s.dev)
        new_off[1:] = torch.cumsum(n[:, 0] + 1, 0)
        s.appended.append((new, new_off))
        sd.sd_index_append(s.ctx, s.slots, new, new_off)
        pos += n + 1
        sd.sd_speculate(s.ctx, s.slots, s.out)


def prepare(case, seed):
    streams = _Streams(case, seed)
    docs, doc_off = streams.corpus(case["corpus"])
    batches = []
    for _ in range(case["rounds"]):
        lens = torch.full((case["new_docs"],), case["new_len"], dtype=torch.int64, device=streams.dev)
        n = case["new_docs"] * case["new_len"]
        batches.append(streams.sequences(lens, n) + (n,))
    capacity = (case["corpus"] + doc_off.numel() - 1
                + case["rounds"] * case["new_docs"] * (case["new_len"] + 1))
    s = _State(case, capacity, case["batch"])
    s.docs, s.doc_off, s.batches = docs, doc_off, batches
    if case["kind"] != "entropy":
        s.requests, s.request_off, s.slots, s.request_tokens = streams.contexts()
        s.out = s.trees()
    if case["kind"] in ("decode", "draft", "entropy"):
        s.build_global()
    if case["kind"] == "insert":
        s.outs = [s.trees() for _ in range(case["rounds"])]
    if case["kind"] in ("draft", "build", "insert"):
        s.take_requests()
    if case["kind"] == "decode":
        _record(s, streams)
        if case["graph"]:
            _decode(s)  # every kernel is loaded before the capture
            torch.cuda.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph):
                _decode(s)
    torch.cuda.synchronize()
    return s


# ---- one pass --------------------------------------------------------------------------------


def _decode(s):
    B = s.case["batch"]
    calls = s.case["calls"]
    s.take_requests()
    sd.sd_speculate(s.ctx, s.slots, s.out)
    for t in range(s.case["steps"]):
        said, n, path, bonus = s.targets[t], s.accept_len[t], s.accept_path[t], s.bonus[t]
        if calls == "fused":
            sd.sd_accept_append_speculate(s.ctx, s.out, s.slots, said, n, path, bonus)
            continue
        if calls == "two":
            sd.sd_accept_append(s.ctx, s.out, s.slots, said, n, path, bonus)
        else:
            sd.sd_accept(s.ctx, s.out, B, said, n, path, bonus)
            sd.sd_index_append(s.ctx, s.slots, *s.appended[t])
        sd.sd_speculate(s.ctx, s.slots, s.out)


def _drafts(trees):
    return {k: getattr(trees, k) for k in ("n_nodes", "tokens", "parents", "match_len", "source",
                                           "scores", "tree_score", "use_draft")}


def run(state):
    s = state
    kind = s.case["kind"]
    if kind == "entropy":
        return np.array(sd.sd_index_entropy(s.ctx), np.float64)
    if kind == "decode":
        if s.graph is not None:
            s.graph.replay()
        else:
            _decode(s)
        return [_drafts(s.out), s.accept_len, s.accept_path, s.bonus]
    if kind == "draft":
        sd.sd_speculate(s.ctx, s.slots, s.out)
        return _drafts(s.out)
    s.build_global()
    if kind == "build":
        sd.sd_speculate(s.ctx, s.slots, s.out)
        return _drafts(s.out)
    for (tokens, off, n), out in zip(s.batches, s.outs):
        sd.sd_index_insert(s.ctx, tokens, off, n)
        sd.sd_speculate(s.ctx, s.slots, out)
    return [_drafts(out) for out in s.outs]


def work(case):
    """Bytes that a pass has to read and write once; there is no floating-point work to speak of."""
    nodes = int(math.floor(case["alpha"] * case["P"]))
    B = case["batch"]
    contexts = 4 * B * case["ctx"] * (5 / 8 if case["ragged"] else 1)
    drafts = B * (16 * nodes + 28)
    index = 12 * case["corpus"]  # tokens in, text and order of the suffixes out
    if case["kind"] == "decode":
        step = B * (4 * (nodes + 1) + 4 * nodes + 8)  # the target's tokens in, acceptance out
        return {"bytes": contexts + drafts + case["steps"] * (step + drafts), "flops": 0}
    if case["kind"] == "draft":
        return {"bytes": contexts + drafts, "flops": 0}
    if case["kind"] == "build":
        return {"bytes": index + contexts + drafts, "flops": 0}
    if case["kind"] == "insert":
        new = 12 * case["new_docs"] * case["new_len"]
        # an insertion moves the order of the old suffixes: read and written once
        return {"bytes": index + contexts + case["rounds"] * (new + 8 * case["corpus"] + drafts),
                "flops": 0}
    return {"bytes": 8 * case["corpus"] + 16, "flops": 0}


def tolerance(case):
    """Trees, tokens and lengths are whole numbers and stay the same; scores are binary64 products
    of quotients, the entropy a binary64 sum over all nodes in whatever order they finish."""
    if case["kind"] == "entropy":
        return {"rel": 1e-9, "max": 1e-9}
    return {"rel": 1e-12, "max": 1e-12}

"""The calls whose speed counts for a user of this framework, as cases that can be timed.

A case is one of these uses of the public entry points (``"kind"``):

``turn``     one generation round of a small live batch: one ``sam_batch_step`` call.  When the
             generated part of the inputs is used up, the sequences are recycled with
             ``sam_batch_reset``, as a server does.
``serve``    the life of a batch of requests: ``sam_batch_reset`` with the new prompts, then every
             generation round until they are done (a ``StepPlan`` over the rounds).
``tree``     the same with a tree draft (``sam_batch_tree_draft``) after every round.
``replay``   the same with all rounds in one ``sam_batch_replay`` call (offline replay of a log).
``prefill``  new prompts for some sequences of a live batch (continuous batching), their first draft
             (a round in which no sequence has accepted tokens), and what state they are in.
``open``     a new batch (``sam_batch_init``), its first draft, its state, and its release.
``build``    the corpus automaton from the corpus tokens (``sam_build``) and the table of its states.

Token streams come from ``paper_2411_10666_amd.synth``: Zipf tokens, parts of which are copies of
corpus or prompt spans.  Everything a pass returns is a whole number and has to stay the same,
but for the probabilities of tree drafts (one float product per edge, rounded once).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2411_10666_amd import binding as sam
from paper_2411_10666_amd.synth import WorkloadSpec, make_corpus, make_workload

# What a case holds unless it says otherwise: corpus tokens (0: none), vocabulary, Zipf exponent,
# copied share of the corpus and of the sequences, mean length of a copy, sequences, prompt tokens
# (drawn from 1 .. prompt for each sequence if ragged), generated tokens, accepted tokens per round
# at most, draft tokens, the paper's l_bias and l_threshold (-1: no auxiliary drafter).
_DEFAULTS = dict(corpus=0, vocab=32000, zipf=1.1, corpus_copy=0.3, seq_copy=0.5, span=20.0, batch=1,
                 prompt=256, ragged=False, gen=0, accept=8, draft=16, bias=0, threshold=-1)


def listed():
    return [
        # one user at a time: a round of one sequence, the smallest call there is
        dict(name="one sequence", kind="turn", corpus=100_000, batch=1, prompt=256, gen=768),
        # the smallest benchmark workload in full
        dict(name="small batch", kind="serve", corpus=100_000, batch=8, prompt=256, gen=768),
        # an ordinary server: the second benchmark workload, its corpus cut so that it builds quickly
        dict(name="ordinary batch", kind="serve", corpus=4_000_000, batch=64, prompt=2048, gen=2048),
        # more sequences, short prompts and long answers: the third benchmark workload's shapes
        dict(name="long answers", kind="serve", corpus=4_000_000, zipf=1.05, corpus_copy=0.4, span=32.0,
             batch=256, prompt=1024, gen=4096, accept=12, draft=24),
        # summarising and question answering over long prompts, no corpus: the fourth one in full
        dict(name="long prompts", kind="serve", batch=1024, prompt=6000, gen=2048, seq_copy=0.7, span=24.0,
             accept=16, draft=32),
        # the largest: the fifth benchmark workload's shapes, large vocabulary
        dict(name="largest batch", kind="serve", corpus=6_000_000, vocab=128256, corpus_copy=0.35, span=40.0,
             batch=1024, prompt=2048, gen=4096, accept=16, draft=32),
        # contexts beyond the 16-bit tables, few sequences
        dict(name="long context", kind="serve", corpus=300_000, batch=12, prompt=40_001, gen=1024, accept=16,
             draft=40, bias=5, threshold=5),
        # requests that join a running batch: ragged prompts for an odd number of its sequences
        dict(name="joining requests", kind="prefill", corpus=1_000_000, batch=256, joining=77, prompt=3000,
             ragged=True, gen=256, accept=8, draft=16),
        # a batch set up for one job: allocation, ragged prompts, first draft
        dict(name="new batch", kind="open", corpus=500_000, batch=48, prompt=1999, ragged=True, gen=512),
        # tree drafts with the paper's draft size and its settings beside an auxiliary drafter
        dict(name="tree drafts", kind="tree", corpus=1_000_000, batch=256, prompt=512, gen=512, top_k=4,
             entries=40, bias=5, threshold=5),
        # a recorded log replayed offline
        dict(name="replayed log", kind="replay", corpus=1_000_000, batch=512, prompt=700, ragged=True, gen=1500,
             accept=12, draft=24),
        # the corpus automaton, as rebuilt whenever the corpus changes
        dict(name="corpus", kind="build", corpus=700_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["turn", "serve", "serve", "serve", "serve", "tree", "replay", "prefill", "open", "build"])
    c = dict(kind=kind, vocab=_log_int(rng, 300, 160_000), zipf=round(rng.uniform(1.0, 1.2), 3),
             corpus_copy=round(rng.uniform(0.2, 0.5), 3), span=round(rng.uniform(8.0, 48.0), 1))
    if kind == "build":
        c["corpus"] = _log_int(rng, 20_000, 700_000)
        return c
    # every fifth batch works without a corpus (a tree draft needs one)
    c["corpus"] = 0 if kind != "tree" and rng.random() < 0.2 else _log_int(rng, 20_000, 2_000_000)
    c["batch"] = _log_int(rng, 1, 8 if kind == "turn" else 1024)
    most = min(50_000, 4_000_000 // c["batch"])          # tokens of a sequence
    c["prompt"] = _log_int(rng, 30, most * 3 // 4)
    c["ragged"] = rng.random() < 0.5
    c["gen"] = _log_int(rng, 60, min(3000, most // 4))
    c["accept"] = rng.randint(1, 24)
    c["gen"] = min(c["gen"], 400 * c["accept"])          # some hundred rounds at most
    c["draft"] = rng.randint(4, 64)
    c["seq_copy"] = round(rng.uniform(0.3, 0.8), 3)
    c["bias"], c["threshold"] = rng.choice([(0, -1), (5, 5)])
    if kind == "tree":
        c["top_k"], c["entries"] = rng.randint(1, 8), rng.randint(8, 80)
    if kind == "prefill":
        c["joining"] = rng.randint(1, c["batch"])
    return c


def _spec(c, seed):
    c = {**_DEFAULTS, **c}
    return WorkloadSpec("case", c["corpus"], c["vocab"], c["zipf"], c["corpus_copy"] if c["corpus"] else 0.0,
                        c["span"], c["batch"], c["prompt"], c["gen"], c["seq_copy"], c["span"], c["accept"],
                        c["draft"], c["bias"], seed)


def _cut(w, c, seed):
    """The prompts back to back and their offsets; ragged ones keep 1 .. prompt of their last tokens."""
    n = np.full(c["batch"], c["prompt"], dtype=np.int64)
    if c["ragged"]:
        n = np.random.default_rng([seed, 100]).integers(1, c["prompt"] + 1, size=c["batch"])
    flat = np.concatenate([w.prompts[b, c["prompt"] - n[b]:] for b in range(c["batch"])])
    return flat, np.concatenate([[0], np.cumsum(n)])


def _rounds(c):
    return max(1, round(2 * c["gen"] / (1 + c["accept"])))


class _State:
    pass


def prepare(case, seed):
    c = {**_DEFAULTS, **case}
    s = _State()
    s.kind = c["kind"]
    spec = _spec(c, seed)
    if s.kind == "build":
        s.tokens, s.vocab = make_corpus(spec), c["vocab"]
        s.states = np.full((3, 2 * c["corpus"]), -1, dtype=np.int32)      # the most that there can be
        return s
    w = make_workload(spec)
    dev = torch.device("cuda")
    s.corpus = sam.sam_build(w.corpus, c["vocab"]) if c["corpus"] else None
    if s.kind == "tree":
        sam.sam_corpus_build_topk(s.corpus, c["top_k"])
    flat, offs = _cut(w, c, seed)
    s.prompts, s.offsets = torch.from_numpy(flat).to(dev), torch.from_numpy(offs).to(dev)
    B, A, L = c["batch"], c["accept"], c["draft"]
    s.sizes = (B, c["vocab"], c["prompt"] + c["gen"], A, L, c["bias"])
    i32 = dict(dtype=torch.int32, device=dev)
    s.threshold = c["threshold"]
    if s.kind in ("open", "prefill"):
        rounds = 1
        s.accepted, s.counts = torch.zeros(1, B, A, **i32), torch.zeros(1, B, **i32)
    else:
        # as many rounds as a sequence takes on average (the number that all are done after depends
        # on the draw): some sequences have finished and feed nothing, some are cut off
        rounds = _rounds(c)
        accepted, counts = np.zeros((rounds, B, A), dtype=np.int32), np.zeros((rounds, B), dtype=np.int32)
        n = min(rounds, w.steps)
        accepted[:n], counts[:n] = w.accepted[:n], w.counts[:n]
        s.accepted, s.counts = torch.from_numpy(accepted).to(dev), torch.from_numpy(counts).to(dev)
    s.match_len, s.draft_len, s.source = (torch.zeros(rounds, B, **i32) for _ in range(3))
    s.draft = torch.zeros(rounds, B, L, **i32)
    s.rounds, s.at = rounds, 0
    if s.kind in ("open", "prefill"):
        s.cursors, s.lengths = torch.zeros(4, B, **i32), torch.zeros(3, B, **i32)
    if s.kind == "open":
        return s
    s.batch = sam.sam_batch_init(s.corpus, s.prompts, s.offsets, *s.sizes)
    sam.sam_batch_set_threshold(s.batch, s.threshold)
    s.slots = torch.arange(B, **i32)
    if s.kind == "prefill":
        # the requests that join: prompts of other sequences, for sequences spread over the batch
        r = np.random.default_rng([seed, 101])
        slots, n = np.sort(r.permutation(B)[:c["joining"]]), np.diff(offs)
        take = r.permutation(B)[:c["joining"]]
        s.slots = torch.from_numpy(slots.astype(np.int32)).to(dev)
        s.prompts = torch.from_numpy(np.concatenate([flat[offs[b]:offs[b + 1]] for b in take])).to(dev)
        s.offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(n[take])])).to(dev)
    if s.kind == "serve":
        s.plan = sam.StepPlan(s.batch, s.accepted, s.counts, s.match_len, s.draft, s.draft_len, s.source)
    if s.kind == "tree":
        s.entries = c["entries"]
        s.tokens, s.parents = (torch.zeros(rounds, B, s.entries, **i32) for _ in range(2))
        s.probs = torch.zeros(rounds, B, s.entries, dtype=torch.float32, device=dev)
        s.tree_sizes = torch.zeros(rounds, B, **i32)
    return s


def _step(s, batch, i):
    sam.sam_batch_step(batch, s.accepted[i], s.counts[i], s.match_len[i], s.draft[i], s.draft_len[i], s.source[i])


def _first_draft(s, batch):
    _step(s, batch, 0)
    sam.sam_batch_debug(batch, *s.cursors)
    sam.sam_batch_sizes(batch, *s.lengths)
    return s.match_len, s.draft, s.draft_len, s.source, s.cursors, s.lengths


def run(s):
    if s.kind == "build":
        corpus = sam.sam_build(s.tokens, s.vocab)
        for row, values in zip(s.states, sam.sam_corpus_export(corpus)):
            row[:values.size] = values
        return s.states
    if s.kind == "open":
        return _first_draft(s, sam.sam_batch_init(s.corpus, s.prompts, s.offsets, *s.sizes))
    if s.kind == "turn":
        if s.at == s.rounds:
            sam.sam_batch_reset(s.batch, s.slots, s.prompts, s.offsets)
            s.at = 0
        i, s.at = s.at, s.at + 1
        _step(s, s.batch, i)
        return s.match_len[i], s.draft[i], s.draft_len[i], s.source[i]
    sam.sam_batch_reset(s.batch, s.slots, s.prompts, s.offsets)
    if s.kind == "prefill":
        return _first_draft(s, s.batch)
    if s.kind == "replay":
        sam.sam_batch_replay(s.batch, s.accepted, s.counts, s.match_len, s.draft, s.draft_len, s.source)
    elif s.kind == "tree":
        for i in range(s.rounds):
            _step(s, s.batch, i)
            sam.sam_batch_tree_draft(s.batch, s.entries, s.tokens[i], s.parents[i], s.probs[i], s.tree_sizes[i])
        return (s.match_len, s.draft, s.draft_len, s.source, s.tokens, s.parents, s.probs, s.tree_sizes)
    else:
        s.plan.run(0, s.rounds)
    return s.match_len, s.draft, s.draft_len, s.source


def work(case):
    """Bytes of one pass.  A token that is fed: itself read and appended to the sequence's text
    (8 B), one transition of each automaton that is there (16 B each), one new state (16 B).  A draft
    token is read and written (8 B); a sequence-round has a count and three results (16 B); an
    entry of a tree draft is read and written with its parent and probability (24 B).  The corpus
    automaton: the tokens (4 B), about 1.4 states a token (32 B)."""
    c = {**_DEFAULTS, **case}
    if c["kind"] == "build":
        return {"bytes": c["corpus"] * (4 + 1.4 * 32) + 8 * c["vocab"], "flops": 0}
    token = 8 + 16 + 16 + (16 if c["corpus"] else 0)
    prompt = (c["prompt"] + 1) / 2 if c["ragged"] else c["prompt"]
    per_round = c["batch"] * (8 * c["draft"] + 16)
    if c["kind"] == "turn":
        return {"bytes": c["batch"] * c["gen"] / _rounds(c) * token + per_round, "flops": 0}
    if c["kind"] == "open":
        return {"bytes": c["batch"] * prompt * token + per_round, "flops": 0}
    if c["kind"] == "prefill":
        return {"bytes": c["joining"] * prompt * token + per_round, "flops": 0}
    if c["kind"] == "tree":
        per_round += c["batch"] * 24 * c["entries"]
    return {"bytes": c["batch"] * (prompt + c["gen"]) * token + _rounds(c) * per_round, "flops": 0}


def tolerance(case):
    """All whole numbers, but for the probabilities of tree drafts: products of at most 80 floats, each
    rounded once in the same order everywhere, so the same bits too; four roundings are allowed."""
    return {"rel": 5e-7} if case["kind"] == "tree" else "exact"

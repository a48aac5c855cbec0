"""Prompts taken whole (one workgroup builds a sequence's automaton) against the CPU
checker: state ids, links, lengths, transitions (through the steps that follow), bit-exact."""
import numpy as np
import pytest

from parity_util import assert_same, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _text(kind, n, vocab, rng):
    x = np.minimum((vocab * rng.random(n) ** 5).astype(np.int64), vocab - 1).astype(np.int32)
    if kind == "copies":
        i = 20
        while i < n:
            k = int(rng.integers(1, 80))
            s = int(rng.integers(0, i))
            k = min(k, i - s, n - i)
            x[i:i + k] = x[s:s + k]
            i += k + int(rng.integers(0, 40))
    elif kind == "one token":
        x[:] = vocab - 1
    elif kind == "periodic":
        x = np.resize(x[:7], n).astype(np.int32)
        x[n // 2] = vocab - 1
    elif kind == "every other":                    # one large group of ever new pairs
        x = (np.arange(n) // 2 % vocab).astype(np.int32)
        x[::2] = 0
    return x


def _compare(prompts, vocab, T, mode, corpus=None, steps=3, A=12, L=20):
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(len(prompts[0]))
    B = len(prompts)
    acc = np.stack([[np.resize(p[len(p) // 3:], (steps, A))[s] if len(p) else np.zeros(A, np.int32)
                     for p in prompts] for s in range(steps)]).astype(np.int32)
    acc[:, :, 5] = rng.integers(0, vocab, size=(steps, B))
    cnt = rng.integers(0, A + 1, size=(steps, B)).astype(np.int32)
    try:
        sam.sam_set_layout_override(mode)
        g, status, _ = run_gpu(corpus, vocab, prompts, acc, cnt, T, A, L)
    finally:
        sam.sam_set_layout_override(0)
    assert status == 0
    r, _ = run_oracle(corpus, prompts, acc, cnt, A, L)
    assert_same(g, r, has_static=corpus is not None)


# around the shortest prompt taken whole, a workgroup's threads, below and above the most whose arrays
# fit into LDS (6144 tokens; its very edge is test_the_most_that_fits_into_lds), the compact
# tables' limit and beyond
@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1024, 1025, 2049, 6000, 6200, 6260, 9001, 16300, 16400, 23456])
@pytest.mark.parametrize("kind,vocab", [("zipf", 32000), ("copies", 500), ("copies", 2)])
def test_sizes(n, kind, vocab):
    rng = np.random.default_rng(n)
    prompts = [_text(kind, k, vocab, rng) for k in (n, n, 1, n // 2 + 1, 0, n - 1, 40)]
    corpus = _text("copies", 3000, vocab, rng)
    corpus[500:1500] = np.resize(prompts[0][-900:], 1000)   # a match far longer than the first window
    _compare(prompts, vocab, n + 40, 0, corpus)


# prompts on both sides of the limit in one launch: 6144 tokens in LDS, 6145 in the sequence's tables
@pytest.mark.parametrize("mode,vocab", [(0, 500), (1, 500), (0, 160000)])
def test_the_most_that_fits_into_lds(mode, vocab):
    rng = np.random.default_rng(mode)
    prompts = [_text("copies", k, vocab, rng) for k in (6143, 6144, 6145, 6146, 6144, 300)]
    _compare(prompts, vocab, 6200, mode, _text("copies", 3000, vocab, rng))
    _compare([prompts[1], prompts[0]], vocab, 6200, mode)            # all in LDS


# the wide tables' working arrays at their largest: every level of names, the longest prompt taken
# whole and one token more (token by token)
@pytest.mark.parametrize("n", [40_001, 65_537, 131_073, 262_144, 262_145])
@pytest.mark.parametrize("kind", ["long copies", "one period"])
def test_long_prompts(n, kind):
    rng = np.random.default_rng(n)
    x = rng.integers(0, 3000, size=n, dtype=np.int32)
    if kind == "one period":
        x = np.resize(x[:200], n).astype(np.int32)
        x[n // 2] = 2999
    else:
        i = 20
        while i < n:
            k = int(min(rng.integers(1, 70_000), i, n - i))
            s = int(rng.integers(0, i - k + 1))
            x[i:i + k] = x[s:s + k]
            i += k + int(rng.integers(1, 40))
    _compare([x, x[:n // 3]], 3000, n + 40, 0)


@pytest.mark.parametrize("kind", ["one token", "periodic", "every other"])
@pytest.mark.parametrize("n", [700, 6100, 6400, 17001])
def test_degenerate_texts(kind, n):
    rng = np.random.default_rng(n)
    _compare([_text(kind, n, 9000, rng)] * 2, 9000, n + 36, 0)


# forced wide, tight slot tables (too small to build in: the serial kernel), C++ loops, large vocabulary
@pytest.mark.parametrize("mode,vocab", [(1, 700), (2, 700), (3, 700), (4, 700), (5, 700), (0, 160000)])
@pytest.mark.parametrize("n", [300, 6500])
def test_layouts(mode, vocab, n):
    rng = np.random.default_rng(mode)
    prompts = [_text("copies", k, vocab, rng) for k in (n, n // 3, 77)]
    _compare(prompts, vocab, n + 40, mode, _text("copies", 2000, vocab, rng))


# small workgroups: more prompts than compute units (up to 512 tokens) and than twice as many
# (up to 1024), and one past either length; ragged, with and without a corpus
@pytest.mark.parametrize("batch,n", [(257, 64), (270, 512), (270, 513), (513, 65), (520, 1024), (520, 1025)])
@pytest.mark.parametrize("mode,with_corpus", [(0, True), (1, False)])
def test_many_prompts(batch, n, mode, with_corpus):
    rng = np.random.default_rng(batch + n)
    sizes = np.concatenate([[n, n - 1, 0, 1, 63, 256, 257], rng.integers(1, n + 1, size=batch)])[:batch]
    prompts = [_text("copies", min(int(k), n), 300, rng) for k in sizes]
    corpus = _text("copies", 3000, 300, rng) if with_corpus else None
    _compare(prompts, 300, n + 40, mode, corpus)


# as many prompts as compute units, the walks over the corpus beside them (small workgroups up to 256
# tokens); more than five for each (token by token up to 87 tokens), all but two of them short
# (up to 94)
@pytest.mark.parametrize("batch,n", [(250, 256), (250, 257), (1300, 87), (1300, 88), (3000, 94), (3000, 96)])
def test_lines_of_the_dispatch(batch, n):
    rng = np.random.default_rng(batch + n)
    sizes = rng.integers(1, n + 1, size=batch) if batch < 2000 else rng.integers(1, 30, size=batch)
    sizes[[3, 77]] = n, n - 1
    corpus = _text("copies", 3000, 300, rng)
    prompts = [_text("copies", int(k), 300, rng) for k in sizes]
    for p in prompts[::9]:
        k = min(len(p), 60)
        p[len(p) - k:] = corpus[700:700 + k]
    _compare(prompts, 300, n + 40, 0, corpus)


@pytest.mark.parametrize("at", [0, 1, 99, 299])
def test_a_bad_token_ends_its_prompt(at):
    """sam_batch_reset with a token outside the vocabulary: the prompt ends in front of it."""
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(at)
    vocab, n = 50, 300
    corpus = _text("copies", 1000, vocab, rng)
    prompts = [_text("copies", n, vocab, rng) for _ in range(3)]
    dev = torch.device("cuda")
    c = sam.sam_build(corpus, vocab)
    offs = torch.arange(4, dtype=torch.int64, device=dev) * n
    flat = np.concatenate(prompts)
    batch = sam.sam_batch_init(c, torch.from_numpy(flat).to(dev), offs, 3, vocab, n + 10, 4, 4, 0)
    bad = flat.copy()
    bad[n + at] = vocab
    sam.sam_batch_reset(batch, torch.arange(3, dtype=torch.int32, device=dev), torch.from_numpy(bad).to(dev), offs)
    assert sam.sam_batch_status(batch) == sam.SAM_STATUS_TOKEN
    out = [torch.empty(3, dtype=torch.int32, device=dev) for _ in range(7)]
    sam.sam_batch_debug(batch, *out[:4])
    sam.sam_batch_sizes(batch, *out[4:])
    got = np.stack([t.cpu().numpy() for t in out], axis=1)
    r, _ = run_oracle(corpus, [prompts[0], prompts[1][:at], prompts[2]], np.zeros((1, 3, 4), np.int32),
                      np.zeros((1, 3), np.int32), 4, 4)
    assert np.array_equal(got[:, :4], r[0]["cursors"])
    assert np.array_equal(got[:, 4:], r[0]["sizes"])


# The static cursor after a prompt: its end occurs in the corpus with `match` tokens and no more
# (around the first window, its double, half the prompt, all of it), once, or first with fewer in
# front of it (the first occurrence then says too little, several times over), or at the very start
@pytest.mark.parametrize("n", [49, 65, 130, 700])
@pytest.mark.parametrize("how", ["once", "shorter first", "at the start"])
def test_matches_at_the_end(n, how):
    rng = np.random.default_rng(n)
    vocab = 3000
    matches = sorted({m for m in (0, 1, 46, 47, 48, 49, 50, 94, 95, 96, 97, 98, 191, 193, 400, n // 2 - 1, n // 2,
                                  n // 2 + 1, n - 2, n - 1, n) if 0 <= m <= n})
    prompts, parts = [], [rng.integers(0, vocab, size=300, dtype=np.int32)]
    for m in matches:
        p = rng.integers(0, vocab, size=n, dtype=np.int32)
        prompts.append(p)
        pieces = [k for k in (48, 49, 55, 100, 210, 430) if k < m] if how == "shorter first" else []
        for k in pieces + [m]:
            parts += [p[n - k:], rng.integers(0, vocab, size=7, dtype=np.int32)]
    if how == "at the start":
        parts = [prompts[-1]] + parts
    _compare(prompts, vocab, n + 40, 0, np.concatenate(parts))


# a few prompts beyond LDS among many short ones, first and last among them (the whole chip builds those alone,
# found through a list), too many to be few, and so much text in the others that one workgroup each builds
# them; then again for some sequences of the batch, in another order
@pytest.mark.parametrize("T,longest", [(9040, 7000), (9040, 9000), (20_040, 20_000)])
@pytest.mark.parametrize("batch,many,short", [(200, 4, 60), (150, 40, 30), (1100, 3, 5500), (3, 2, 10)])
def test_few_long_prompts(T, longest, batch, many, short):
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(batch)
    vocab = 300
    lengths = rng.integers(0, short + 1, size=batch)
    lengths[rng.permutation(batch)[:many]] = rng.integers(6145, longest, size=many)
    lengths[0], lengths[-1] = longest, 6145
    pool = _text("copies", 60_000, vocab, rng)
    prompts = [pool[a:a + n] for a, n in zip(rng.integers(0, 60_000 - lengths), lengths)]
    if batch * short < 1_000_000:
        _compare(prompts, vocab, T, 0, _text("copies", 2000, vocab, rng))
    dev = torch.device("cuda")
    take = rng.permutation(batch)[:batch * 3 // 4 + 1]
    order = rng.permutation(take)
    again = [np.concatenate([prompts[i], [vocab]]).astype(np.int32) if k % 3 == 0 else prompts[i]
             for k, i in enumerate(take)]              # every third one ends in a bad token
    again = [p if len(p) <= T else p[:T] for p in again]

    def flat(ps):
        return (torch.from_numpy(np.concatenate(ps)).to(dev),
                torch.from_numpy(np.cumsum([0] + [len(p) for p in ps])).to(dev))

    seen = []
    for mode in (0, 128):
        try:
            sam.sam_set_layout_override(mode)
            b = sam.sam_batch_init(None, *flat(prompts), batch, vocab, T, 4, 4)
        finally:
            sam.sam_set_layout_override(0)
        sam.sam_batch_reset(b, torch.from_numpy(order.astype(np.int32)).to(dev), *flat(again))
        out = [torch.zeros(batch, dtype=torch.int32, device=dev) for _ in range(8)]
        draft = torch.zeros(batch, 4, dtype=torch.int32, device=dev)
        row = torch.from_numpy(np.stack([pool[i:i + 4] for i in range(batch)])).to(dev)
        sam.sam_batch_step(b, row, torch.full_like(out[0], 4), out[0], draft, out[1], out[2])
        sam.sam_batch_debug(b, None, None, *out[3:5])
        sam.sam_batch_sizes(b, *out[5:])
        assert sam.sam_batch_status(b) == sam.SAM_STATUS_TOKEN
        seen.append(torch.cat([torch.stack(out).flatten(), draft.flatten()]).cpu())
        del b
    assert torch.equal(*seen)


# a captured init, replayed with prompts of other lengths in the same buffers: longer ones than it was
# captured with, within and beyond what LDS holds, in tables with room for the working arrays and without;
# captured beyond LDS (the whole chip's launches are in the graph): shorter ones, the same and longer ones
@pytest.mark.parametrize("captured,replayed,T", [(100, 300, 340), (100, 2500, 2600), (2000, 9000, 9040),
                                                 (70, 20_000, 20_040), (30, 500, 540),
                                                 (9000, 14_900, 15_000), (9000, 8000, 15_000),
                                                 (20_000, 30_000, 30_040), (14_000, 100_000, 100_040)])
def test_replayed_init_takes_longer_prompts(captured, replayed, T):
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(captured)
    vocab, B, A, L = 400, 2, 8, 8
    corpus = _text("copies", 2000, vocab, rng)
    c = sam.sam_build(corpus, vocab)
    dev = torch.device("cuda")
    first = [_text("copies", n, vocab, rng) for n in (captured, captured // 2)]
    tokens = torch.zeros(2 * replayed, dtype=torch.int32, device=dev)
    offsets = torch.zeros(B + 1, dtype=torch.int64, device=dev)

    def put(prompts):
        flat = np.concatenate(prompts)
        tokens[:len(flat)].copy_(torch.from_numpy(flat))
        offsets.copy_(torch.from_numpy(np.cumsum([0] + [len(p) for p in prompts])))
        torch.cuda.synchronize()

    put(first)
    offs = offsets.cpu().numpy()
    del_me = sam.sam_batch_init_noalloc(c, tokens, offsets, offs, B, vocab, T, A, L)      # looks the buffer up
    del del_me
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        batch = sam.sam_batch_init_noalloc(c, tokens, offsets, offs, B, vocab, T, A, L, 0, stream)
    i32 = dict(dtype=torch.int32, device=dev)
    zero = np.zeros((1, B, A), np.int32), np.zeros((1, B), np.int32)
    accepted, counts = (torch.from_numpy(z[0]).to(dev) for z in zero)
    for prompts in (first, [_text("copies", n, vocab, rng) for n in (replayed // 3, replayed)],
                    [_text("copies", n, vocab, rng) for n in (replayed, 5)], first):
        put(prompts)
        graph.replay()
        torch.cuda.synchronize()
        ml, dl, src = (torch.empty(B, **i32) for _ in range(3))
        dr = torch.empty(B, L, **i32)
        state = [torch.empty(B, **i32) for _ in range(7)]
        sam.sam_batch_step(batch, accepted, counts, ml, dr, dl, src)
        sam.sam_batch_debug(batch, *state[:4])
        sam.sam_batch_sizes(batch, *state[4:])
        assert sam.sam_batch_status(batch) == 0
        g = dict(match_len=ml, draft_len=dl, source=src, draft=dr, cursors=torch.stack(state[:4], 1),
                 sizes=torch.stack(state[4:], 1))
        r, _ = run_oracle(corpus, prompts, *zero, A, L)
        assert_same([{k: v.cpu().numpy() for k, v in g.items()}], r)
    del batch

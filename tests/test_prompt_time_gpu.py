"""A prompt taken whole is not slower than the same tokens fed one by one (to empty sequences,
through sam_batch_step), for texts that are hard on the whole build, and a corpus built on the device is
not slower than on the host.  Both are measured here, on
the same device, the shortest of several runs each; the build takes two thirds of the time at most."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _shortest(f, runs=7):
    import torch
    best = float("inf")
    for _ in range(runs):
        torch.cuda.synchronize()
        start = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - start)
    return best


def _whole_and_one_by_one(prompts, corpus, vocab):
    """All prompts have the same length."""
    import torch
    from paper_2411_10666_amd import binding as sam
    dev = torch.device("cuda")
    B, n = prompts.shape
    A = next(a for a in range(4096, 0, -1) if n % a == 0)
    i32 = dict(dtype=torch.int32, device=dev)
    flat = torch.from_numpy(prompts.reshape(-1)).to(dev)
    offsets = torch.arange(B + 1, dtype=torch.int64, device=dev) * n
    nothing = torch.zeros(B + 1, dtype=torch.int64, device=dev)
    slots = torch.arange(B, **i32)
    rows = torch.from_numpy(np.ascontiguousarray(prompts.reshape(B, n // A, A).transpose(1, 0, 2))).to(dev)
    counts = torch.full((B,), A, **i32)
    out = torch.empty(B, **i32), torch.empty(B, 4, **i32), torch.empty(B, **i32), torch.empty(B, **i32)
    c = sam.sam_build(corpus, vocab) if corpus is not None else None
    batch = sam.sam_batch_init(c, flat, nothing, B, vocab, n + 8, A, 4, 0)
    states = []

    def state():
        s = [torch.empty(B, **i32) for _ in range(7)]
        sam.sam_batch_debug(batch, *s[:4])
        sam.sam_batch_sizes(batch, *s[4:])
        states.append(torch.stack(s)[(0 if c is not None else 2):].cpu().numpy())

    def one_by_one():
        sam.sam_batch_reset(batch, slots, flat, nothing)
        for row in rows:
            sam.sam_batch_step(batch, row, counts, *out)

    slow = _shortest(one_by_one)
    state()
    fast = _shortest(lambda: sam.sam_batch_reset(batch, slots, flat, offsets))
    state()
    assert np.array_equal(*states)
    print("%d x %d: whole %.0f us, one by one %.0f us" % (B, n, fast * 1e6, slow * 1e6), flush=True)
    return fast, slow


@pytest.mark.parametrize("kind", ["equal tokens", "run, then another", "left padding", "period of two"])
@pytest.mark.parametrize("batch,n", [(1, 1000), (64, 6000), (64, 9000)])
def test_repeating_texts(kind, batch, n):
    rng = np.random.default_rng(n)
    x = np.full((batch, n), 7, np.int32)
    if kind == "run, then another":
        x[:, -1] = 9
    elif kind == "left padding":
        x[:, n * 3 // 4:] = rng.integers(0, 500, size=(batch, n - n * 3 // 4))
    elif kind == "period of two":
        x[:, ::2] = 3
        x[:, -1] = 9
    fast, slow = _whole_and_one_by_one(x, None, 500)
    assert fast < slow


@pytest.mark.parametrize("n,period", [(200_000, 134), (262_144, 512), (262_144, 60)])
def test_long_periodic_texts(n, period):
    rng = np.random.default_rng(n)
    x = np.resize(rng.integers(0, 3000, size=period, dtype=np.int32), (1, n))
    fast, slow = _whole_and_one_by_one(np.ascontiguousarray(x), None, 3000)
    assert fast < slow


@pytest.mark.parametrize("batch,n", [(64, 3073), (256, 3073), (1024, 800), (64, 12_300)])
def test_passages_of_the_corpus(batch, n):
    """Prompts that occur in the corpus as a whole: the walk over the corpus automaton decides."""
    rng = np.random.default_rng(n)
    vocab = 8000
    corpus = np.minimum((vocab * rng.random(2_000_000) ** 4).astype(np.int64), vocab - 1).astype(np.int32)
    starts = rng.integers(0, corpus.size - n, size=batch)
    fast, slow = _whole_and_one_by_one(np.stack([corpus[a:a + n] for a in starts]), corpus, vocab)
    assert fast < slow


@pytest.mark.parametrize("batch", [1, 256])
def test_tree_drafts_with_many_children(batch):
    """A draft's time is its chain of pops, however long the queue: 128 entries of 8 children each
    take little longer than of one child each (1.05 times as long as measured; half as long again allowed)."""
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(1)
    vocab, n, size = 50, 60, 128
    dev = torch.device("cuda")
    corpus = np.minimum((vocab * rng.random(1_000_000) ** 2).astype(np.int64), vocab - 1).astype(np.int32)
    c = sam.sam_build(corpus, vocab)
    flat = torch.from_numpy(corpus[:batch * n].copy()).to(dev)
    out = [torch.empty(batch, size, dtype=d, device=dev) for d in (torch.int32, torch.int32, torch.float32)]
    sizes = torch.empty(batch, dtype=torch.int32, device=dev)
    times = []
    for k in (1, 8):
        sam.sam_corpus_build_topk(c, k)
        b = sam.sam_batch_init(c, flat, torch.arange(batch + 1, dtype=torch.int64, device=dev) * n, batch, vocab,
                               n + 8, 4, 4)
        times.append(_shortest(lambda: sam.sam_batch_tree_draft(b, size, *out, sizes), 30))
        assert int(sizes.min()) == size
        del b
    print("128 entries, k = 1: %.0f us, k = 8: %.0f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 1.5 * times[0]


@pytest.mark.parametrize("kind", ["equal tokens", "period of two", "half equal", "padded documents"])
def test_repeating_corpora(kind):
    """Texts with few large groups, of which one workgroup sorts each (device 0.2 to 0.7 of the host's time as measured)."""
    rng = np.random.default_rng(3)
    n = 700_000
    x = np.full(n, 7, np.int32)
    if kind == "period of two":
        x[::2] = 3
    elif kind == "half equal":
        x[:n // 2] = rng.integers(0, 500, size=n // 2)
    elif kind == "padded documents":
        for at in range(0, n, 4000):
            x[at:at + 500] = rng.integers(0, 500, size=500)
    device, host = _device_and_host(x, 500, 3)
    assert device < host


def _device_and_host(x, vocab, runs):
    from paper_2411_10666_amd import binding as sam
    times = []
    for mode in (0, 128):
        try:
            sam.sam_set_layout_override(mode)
            times.append(_shortest(lambda: sam.sam_build(x, vocab), runs))
        finally:
            sam.sam_set_layout_override(0)
    print("sam_build %.2f ms, on the host %.2f ms" % (times[0] * 1e3, times[1] * 1e3), flush=True)
    return times


# of `part` of the text a period repeats throughout, then comes other text (another token, if it is all)
@pytest.mark.parametrize("n", [12_000, 30_000, 100_000, 200_000, 500_000])
@pytest.mark.parametrize("period,part", [(1, 1), (1, 0.75), (1, 0.5), (2, 1), (3, 1), (20, 1), (150, 1), (700, 1), (20, 0.5)])
def test_repeating_corpora_of_any_size(n, period, part):
    """Where the device is slower at text that repeats, the host builds (1.05 of its time at most as measured, but for one
    text near a line 1.26; without the look at the text up to 2.7)."""
    rng = np.random.default_rng(n)
    x = (500 * rng.random(n) ** 4).astype(np.int32)
    x[:int(n * part)] = np.resize(rng.integers(0, 500, size=period), int(n * part))
    x[-1] = 9
    built, host = _device_and_host(x, 500, 5)
    assert built < 1.5 * host


@pytest.mark.parametrize("kind", ["equal tokens", "period of two", "padding"])
@pytest.mark.parametrize("batch,n", [(1, 6500), (600, 8000)])
def test_many_repeating_prompts(kind, batch, n):
    """Prompts beyond LDS by the whole chip take little longer than by one workgroup each at worst (1.0 of it as
    measured; a quarter more allowed)."""
    rng = np.random.default_rng(n)
    x = np.full(n, 7, np.int32)
    if kind == "period of two":
        x[::2] = 3
    elif kind == "padding":
        x[n * 3 // 4:] = rng.integers(0, 500, size=n - n * 3 // 4)
    chip, workgroups = _chip_and_workgroups([x] * batch)
    assert chip < 1.25 * workgroups


def _chip_and_workgroups(prompts):
    import torch
    from paper_2411_10666_amd import binding as sam
    dev, B = torch.device("cuda"), len(prompts)
    lengths = [len(p) for p in prompts]
    flat = torch.from_numpy(np.concatenate(prompts)).to(dev)
    offsets = torch.from_numpy(np.cumsum([0] + lengths)).to(dev)
    slots = torch.arange(B, dtype=torch.int32, device=dev)
    times = []
    for mode in (0, 128):
        try:
            sam.sam_set_layout_override(mode)
            b = sam.sam_batch_init(None, flat, torch.zeros_like(offsets), B, 32000, max(lengths) + 8, 4, 4)
        finally:
            sam.sam_set_layout_override(0)
        times.append(_shortest(lambda: sam.sam_batch_reset(b, slots, flat, offsets)))
        del b
    print("chip %.0f us, workgroups %.0f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    return times


@pytest.mark.parametrize("batch,short", [(1280, 64), (1280, 2000), (640, 6000)])
@pytest.mark.parametrize("longest", [6500, 100_000])
def test_one_long_prompt_among_short_ones(batch, short, longest):
    """(1.03 as long at most as measured; it was up to 1.7, where the chip's launches covered all prompts)"""
    rng = np.random.default_rng(batch)
    text = np.minimum((32000 * rng.random(longest + short) ** 5).astype(np.int64), 31999).astype(np.int32)
    prompts = [text[:short]] * batch
    prompts[batch // 3] = text[short:]
    chip, workgroups = _chip_and_workgroups(prompts)
    assert chip < 1.15 * workgroups

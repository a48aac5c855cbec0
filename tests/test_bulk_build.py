"""Automata built by the whole chip, phase by phase: corpora against the host builder, prompts too
long for LDS against the oracle (their sizes: test_prompt_gpu.py), everything bit-exact."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from test_sanitizers import FLAGS, ROOT, _have_sanitizer_runtime


def test_phases_under_asan_ubsan(tmp_path):
    """The phases, one after the other on the CPU, over regions of exactly the library's sizes."""
    if not (shutil.which("gcc") and shutil.which("g++")):
        pytest.skip("gcc / g++ not available")
    if not _have_sanitizer_runtime(tmp_path):
        pytest.skip("the sanitizer runtime (libasan / libubsan) is not installed")
    exe = tmp_path / "bulk_build_driver"
    subprocess.check_call(["g++", "-std=c++17", "-pthread"] + FLAGS + [
        os.path.join(ROOT, "tests", "bulk_build_driver.cpp"),
        os.path.join(ROOT, "paper_2411_10666_amd", "csrc", "sam_host.cpp"), "-o", str(exe)])
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0")
    p = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-4000:]
    assert p.stdout.strip().endswith("ok")


def _text(kind, n, vocab, rng):
    x = (rng.random(n) ** 3 * vocab).astype(np.int32)
    if kind == "copies":
        x[n // 2:] = x[:n - n // 2]
        x[n * 3 // 4:] = x[n // 8:n // 8 + n - n * 3 // 4]
    elif kind == "one token":
        x[:] = vocab - 1
        x[-1] = 0
    elif kind == "period":
        x = np.resize(x[:7], n).astype(np.int32)
    return x


def _saved(corpus, path, n, vocab):
    """The bytes of the saved file, its root table and its transitions in order."""
    from paper_2411_10666_amd import binding as sam
    sam.sam_corpus_save(corpus, path)
    raw = open(path, "rb").read()
    at = 64 + 4 * n + 12 * sam.sam_corpus_info(corpus)[0]
    slots = np.frombuffer(raw[at + 8 * vocab:], dtype=np.uint32).reshape(-1, 4)
    used = slots[slots[:, 0] != 0xFFFFFFFF]
    return raw, raw[at:at + 8 * vocab], used[np.lexsort((used[:, 1], used[:, 0]))]


# around a wave, a workgroup's tile (2048), the largest group that is counted (1024: two tokens or one),
# two runs of tiles, the fifth level of minima (32 768) and the size from which sam_build does it by itself
@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 2, 3, 9, 64, 65, 1025, 2047, 2048, 2049, 9999, 10000, 33000, 530_000])
@pytest.mark.parametrize("kind,vocab", [("zipf", 32000), ("zipf", 2), ("copies", 200_000), ("one token", 3),
                                        ("period", 60)])
def test_corpus_like_the_host_builders(tmp_path, n, kind, vocab):
    import torch
    from paper_2411_10666_amd import binding as sam
    x = _text(kind, n, vocab, np.random.default_rng(n))
    host = sam.sam_build_host_only(x, vocab)
    try:
        sam.sam_set_layout_override(64)
        built = [sam.sam_build(x, vocab) for _ in range(2)]
    finally:
        sam.sam_set_layout_override(0)
    torch.cuda.synchronize()
    assert sam.sam_corpus_info(built[0])[:2] == sam.sam_corpus_info(host)[:2]
    for a, b in zip(sam.sam_corpus_export(built[0]), sam.sam_corpus_export(host)):
        assert np.array_equal(a, b)
    raw, root, slots = _saved(built[0], str(tmp_path / "a.sam"), n, vocab)
    again = _saved(built[1], str(tmp_path / "b.sam"), n, vocab)[0]
    _, host_root, host_slots = _saved(host, str(tmp_path / "c.sam"), n, vocab)
    assert raw == again                                  # the same file every time
    assert root == host_root and np.array_equal(slots, host_slots)
    loaded = sam.sam_corpus_load_host_only(str(tmp_path / "a.sam"))
    assert sam.sam_corpus_info(loaded)[:2] == sam.sam_corpus_info(host)[:2]


def _runs(n, run, vocab, rng, token):
    """Runs of one token (of `run` of them, of up to as many, or of one of two lengths) between other text."""
    x = _text("zipf", n, vocab, rng)
    at = int(rng.integers(0, 30))
    while at < n:
        k = run if run > 0 else int(rng.integers(1, -run))
        x[at:at + k] = token
        at += k + int(rng.integers(1, 60))
    return x


# groups beyond 1024 places whose second names are mostly the same: smaller and larger ones from none to more
# than 256 (the most that are counted) and 2048 (a tile), names of up to 2 bytes and of more
@pytest.mark.gpu
@pytest.mark.parametrize("n", [2600, 9000, 66_000])
@pytest.mark.parametrize("run", [1029, 2055, -300, -3000, 257, 50])
@pytest.mark.parametrize("token", [0, 20, 59])
def test_large_groups(n, run, token):
    import torch
    from paper_2411_10666_amd import binding as sam
    vocab = 60
    rng = np.random.default_rng([n, abs(run), token])
    x = _runs(n, run, vocab, rng, token)
    host = sam.sam_build_host_only(x, vocab)
    try:
        sam.sam_set_layout_override(64)
        built = sam.sam_build(x, vocab)
    finally:
        sam.sam_set_layout_override(0)
    assert sam.sam_corpus_info(built)[:2] == sam.sam_corpus_info(host)[:2]
    for a, b in zip(sam.sam_corpus_export(built), sam.sam_corpus_export(host)):
        assert np.array_equal(a, b)
    if n < 6145:
        return
    # as prompts: by the whole chip and by one workgroup each
    prompts = [x, x[:n - 1], x[n // 8:]]
    dev, seen = torch.device("cuda"), []
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum([len(p) for p in prompts])])).to(dev)
    flat = torch.from_numpy(np.concatenate(prompts)).to(dev)
    for mode in (0, 128):
        try:
            sam.sam_set_layout_override(mode)
            batch = sam.sam_batch_init(None, flat, offs, 3, vocab, n + 30, 16, 8, 0)
        finally:
            sam.sam_set_layout_override(0)
        out = [torch.zeros(3, dtype=torch.int32, device=dev) for _ in range(8)]
        draft = torch.zeros(3, 8, dtype=torch.int32, device=dev)
        row = torch.from_numpy(np.stack([p[n // 2:n // 2 + 16] for p in prompts])).to(dev)
        sam.sam_batch_step(batch, row, torch.full_like(out[0], 16), out[0], draft, out[1], out[2])
        sam.sam_batch_debug(batch, None, None, *out[3:5])
        sam.sam_batch_sizes(batch, *out[5:])
        assert sam.sam_batch_status(batch) == 0
        seen.append(torch.cat([torch.stack(out).flatten(), draft.flatten()]).cpu())
    assert torch.equal(*seen)


@pytest.mark.gpu
@pytest.mark.parametrize("vocab,n", [(5, 900), (400, 12_000)])
def test_steps_over_a_corpus_built_on_the_device(vocab, n):
    from parity_util import assert_same, run_gpu, run_oracle
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(n)
    x = _text("copies", n, vocab, rng)
    prompts = [x[k:k + 70].copy() for k in (0, n // 3, n - 70)]
    acc = rng.integers(0, vocab, size=(6, 3, 8)).astype(np.int32)
    acc[:, 0] = np.resize(x[100:], (6, 8))
    cnt = np.full((6, 3), 8, dtype=np.int32)
    try:
        sam.sam_set_layout_override(64)
        corpus = sam.sam_build(x, vocab)
    finally:
        sam.sam_set_layout_override(0)
    g, status, _ = run_gpu(x, vocab, prompts, acc, cnt, 200, 8, 10, gpu_corpus=corpus)
    r, _ = run_oracle(x, prompts, acc, cnt, 8, 10)
    assert status == 0
    assert_same(g, r)


@pytest.mark.gpu
@pytest.mark.parametrize("request_", [1, 2, 3, 4, 5, 6])
def test_no_room_on_the_device_to_build(tmp_path, request_):
    """Whichever device allocation fails (text, root, two for working arrays, transitions, state records), the host
    builds: the file is the one that its builder writes, the corpus serves a batch, and nothing stays behind."""
    import torch
    from parity_util import assert_same, run_gpu, run_oracle
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(request_)
    vocab, n = 400, 300_000
    x = _text("copies", n, vocab, rng)
    prompts = [x[k:k + 70].copy() for k in (0, n // 3, n - 70)]
    acc = np.resize(x[100:], (4, 3, 8)).astype(np.int32)
    cnt = np.full((4, 3), 8, dtype=np.int32)
    torch.cuda.synchronize()
    free = []
    for _ in range(12):
        try:
            sam.sam_set_layout_override(request_ << 8)
            corpus = sam.sam_build(x, vocab)
        finally:
            sam.sam_set_layout_override(0)
        free.append(torch.cuda.mem_get_info()[0])
    # The runtime's own buffers come with the first builds (39 MB seen), then what is free goes to and fro by the 2 MB that
    # it gives out at a time.  The smallest of the arrays that could stay, the text, takes 1.2 MB a build: 9.6 MB in 8.
    assert free[3] - free[11] < 8 << 20
    host = sam.sam_build_host_only(x, vocab)
    assert _saved(corpus, str(tmp_path / "a.sam"), n, vocab)[0] == _saved(host, str(tmp_path / "b.sam"), n, vocab)[0]
    g, status, _ = run_gpu(x, vocab, prompts, acc, cnt, 200, 8, 10, gpu_corpus=corpus)
    r, _ = run_oracle(x, prompts, acc, cnt, 8, 10)
    assert status == 0
    assert_same(g, r)


@pytest.mark.gpu
def test_group_too_large_for_the_device():
    """More than 2^23 positions that end in the same tokens: the device gives up and the host builds."""
    from paper_2411_10666_amd import binding as sam
    n = (1 << 23) + 2000
    corpus = sam.sam_build(np.full(n, 7, dtype=np.int32), 500)
    assert sam.sam_corpus_info(corpus)[:2] == (n + 1, n)
    length, link, endpos = sam.sam_corpus_export(corpus)
    each = np.arange(n + 1)
    assert np.array_equal(length, each) and np.array_equal(link, each - 1) and np.array_equal(endpos, each)
    for state in (0, 1, n - 1):
        assert sam.sam_corpus_find(corpus, state, 7) == state + 1


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["device", "host", "file"])
def test_room_for_the_small_table_is_made(tmp_path, how):
    """The table that the walks look up is asked for while working memory is still held.  Where there is no
    room beside that, it is given back first: the full table does not stay."""
    from parity_util import assert_same, run_gpu, run_oracle
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(4)
    vocab, n = 300, 40_000
    x = _text("copies", n, vocab, rng)
    sam.sam_corpus_save(sam.sam_build_host_only(x, vocab), str(tmp_path / "a.sam"))
    built = []
    for mode in (0, 7 << 8):
        try:
            sam.sam_set_layout_override(mode | (128 if how == "host" else 0))
            built.append(sam.sam_corpus_load(str(tmp_path / "a.sam")) if how == "file" else sam.sam_build(x, vocab))
        finally:
            sam.sam_set_layout_override(0)
    assert sam.sam_corpus_info(built[0]) == sam.sam_corpus_info(built[1])        # the device's bytes too
    prompts = [x[k:k + 70].copy() for k in (0, n // 3, n - 70)]
    acc = np.resize(x[100:], (4, 3, 8)).astype(np.int32)
    cnt = np.full((4, 3), 8, dtype=np.int32)
    g, status, _ = run_gpu(x, vocab, prompts, acc, cnt, 200, 8, 10, gpu_corpus=built[1])
    r, _ = run_oracle(x, prompts, acc, cnt, 8, 10)
    assert status == 0
    assert_same(g, r)


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [-1, 50, 2**31 - 1])
def test_corpus_token_outside_the_vocabulary(bad):
    from paper_2411_10666_amd import binding as sam
    x = np.zeros(30_000, dtype=np.int32)
    x[[12_345, 20_000]] = bad
    said = []
    for mode, build in ((64, sam.sam_build), (0, sam.sam_build), (0, sam.sam_build_host_only)):
        with pytest.raises(sam.SamError) as e:
            try:
                sam.sam_set_layout_override(mode)
                build(x, 50)
            finally:
                sam.sam_set_layout_override(0)
        assert e.value.code == sam.SAM_ETOKEN
        said.append(str(e.value))
    assert said[0] == said[1] == said[2] and "12345" in said[0]


@pytest.mark.gpu
@pytest.mark.parametrize("T,vocab", [(16_366, 300), (30_000, 300)])
def test_long_prompts_cut_at_a_bad_token(T, vocab):
    """Whole-chip builds, one workgroup each (testing mode) and prompts that end in front of the bad token
    leave the same sequences."""
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(T)
    n = T - 3                                            # the most that the 16-bit tables have room for
    prompts = [_text("copies", k, vocab, rng) for k in (n, n - 1, 7000, 6200, 9000, 300)]
    cut = [n, 8000, 0, 1, 6500, 300]
    whole = [np.concatenate([p[:c], [vocab + 5], p[c + 1:]]).astype(np.int32) if c < len(p) else p
             for p, c in zip(prompts, cut)]
    short = [p[:c] for p, c in zip(prompts, cut)]
    dev, seen = torch.device("cuda"), []
    for mode, ps in ((0, whole), (128, whole), (0, short)):
        B = len(ps)
        offs = torch.from_numpy(np.concatenate([[0], np.cumsum([len(p) for p in ps])])).to(dev)
        flat = torch.from_numpy(np.concatenate(ps)).to(dev)
        slots = torch.arange(B, dtype=torch.int32, device=dev)
        try:
            sam.sam_set_layout_override(mode)
            batch = sam.sam_batch_init(None, flat, torch.zeros_like(offs), B, vocab, T, 2, 4, 0)
        finally:
            sam.sam_set_layout_override(0)
        sam.sam_batch_reset(batch, slots, flat, offs)
        out = [torch.zeros(B, dtype=torch.int32, device=dev) for _ in range(10)]
        draft = torch.zeros(B, 4, dtype=torch.int32, device=dev)
        row = torch.full((B, 2), 7, dtype=torch.int32, device=dev)
        sam.sam_batch_step(batch, row, torch.full_like(slots, 2), out[0], draft, out[1], out[2])
        sam.sam_batch_debug(batch, *out[3:7])
        sam.sam_batch_sizes(batch, *out[7:])
        assert sam.sam_batch_status(batch) == (sam.SAM_STATUS_TOKEN if ps is whole else 0)
        seen.append(torch.cat([torch.stack(out[:3] + out[5:]).flatten(), draft.flatten()]).cpu())
    assert torch.equal(seen[0], seen[1]) and torch.equal(seen[0], seen[2])


@pytest.mark.gpu
@pytest.mark.parametrize("T", [(1 << 26) - 2, 1 << 26])
def test_record_tables_around_4_gib(T):
    """The wide layout's assembly has byte offsets of 32 bits: the largest table it takes, and one that is
    left to the compiled loop."""
    from parity_util import assert_same, run_gpu, run_oracle
    rng = np.random.default_rng(3)
    prompts = [_text("copies", 7000, 300, rng)]
    acc = np.resize(prompts[0][3000:], (5, 1, 16)).astype(np.int32)
    acc[:, :, 7] = rng.integers(0, 300, size=(5, 1))
    cnt = np.full((5, 1), 16, dtype=np.int32)
    g, status, _ = run_gpu(None, 300, prompts, acc, cnt, T, 16, 20)
    r, _ = run_oracle(None, prompts, acc, cnt, 16, 20)
    assert status == 0
    assert_same(g, r, has_static=False)


@pytest.mark.gpu
def test_noalloc_batches_with_long_prompts():
    """sam_batch_init_noalloc with prompts beyond LDS (its tables are 32 MB, its calls make no allocation),
    then with short ones, against sam_batch_init."""
    import torch
    from paper_2411_10666_amd import binding as sam
    rng = np.random.default_rng(8)
    dev, T, vocab = torch.device("cuda"), 15_000, 900
    for lengths in ((14_000, 200, 9000), (500, 20, 63)):
        prompts = [_text("copies", n, vocab, rng) for n in lengths]
        offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
        flat, d_offs = torch.from_numpy(np.concatenate(prompts)).to(dev), torch.from_numpy(offs).to(dev)
        seen = []
        for noalloc in (True, False):
            batch = (sam.sam_batch_init_noalloc(None, flat, d_offs, offs, 3, vocab, T, 8, 8) if noalloc
                     else sam.sam_batch_init(None, flat, d_offs, 3, vocab, T, 8, 8))
            out = [torch.zeros(3, dtype=torch.int32, device=dev) for _ in range(10)]
            draft = torch.zeros(3, 8, dtype=torch.int32, device=dev)
            row = torch.from_numpy(np.stack([np.resize(p[5:], 8) for p in prompts])).to(dev)
            sam.sam_batch_step(batch, row, torch.full_like(out[0], 8), out[0], draft, out[1], out[2])
            sam.sam_batch_debug(batch, *out[3:7])
            sam.sam_batch_sizes(batch, *out[7:])
            assert sam.sam_batch_status(batch) == 0
            seen.append(torch.cat([torch.stack(out[:3] + out[5:]).flatten(), draft.flatten()]).cpu())
            del batch
        assert torch.equal(*seen)

"""Appends of many tokens per call against the oracle: the kernel with a thread per new position and
the one with a workgroup per problem, with the buckets and with the fill counts only in LDS, on an
empty and on a filled index."""
import numpy as np
import pytest
import torch

from paper_2503_05330_amd import binding

pytestmark = pytest.mark.gpu


# sizes around a wave (64), a lane's four positions, a workgroup's 256; two symbols: chains of
# hundreds of full buckets
@pytest.mark.parametrize("problems,vocab,query,edits,flags,sizes", [
    (1, 40, 3, 0, binding.MATCH_INDEX, (1, 63, 64, 65, 256, 257)),
    (1, 40, 3, 1, binding.MATCH_INDEX, (2, 64, 65, 300)),
    (1, 40, 6, 1, binding.MATCH_INDEX, (3, 300, 1)),
    (1, 2, 3, 0, binding.MATCH_INDEX, (255, 1, 256)),
    (1, 40, 3, 0, binding.MATCH_SCAN, (1, 65, 257)),
    (24, 40, 3, 0, binding.MATCH_INDEX, (255, 1, 130, 66, 257)),
    (24, 40, 6, 0, binding.MATCH_INDEX, (67, 258, 5, 90)),
    (24, 40, 3, 1, binding.MATCH_INDEX, (254, 253)),
    (24, 40, 6, 1, binding.MATCH_INDEX, (251, 3, 256)),
    (25, 2, 2, 0, binding.MATCH_INDEX, (300, 259)),
])
@pytest.mark.parametrize("ragged", (False, True))
def test_appends_of_many_tokens(oracle, problems, vocab, query, edits, flags, sizes, ragged):
    _appends(oracle, problems, 5, 720, vocab, query, edits, flags, sizes, ragged)


# what takes a workgroup per problem: buckets in LDS (up to 2048 of them), fill counts only (more), grams
# of up to four tokens and longer ones; with counts some problems take less than a posting per bucket.
# (the assertion repeats the library's rule for the first size)
@pytest.mark.parametrize("problems,paths,max_len,query,edits,sizes", [
    (64, 5, 720, 3, 0, (255, 1, 257, 180)),
    (64, 5, 720, 6, 0, (258, 5, 200)),
    (40, 5, 720, 3, 1, (254, 253)),
    (40, 5, 400, 6, 1, (130, 125, 120)),
    (64, 20, 1000, 3, 0, (400, 370)),
    (64, 20, 1000, 6, 0, (370, 361)),
    (40, 8, 800, 3, 1, (300, 290)),
    (40, 5, 720, 6, 1, (251, 3, 256)),
])
@pytest.mark.parametrize("ragged", (False, True))
def test_appends_by_a_workgroup_per_problem(oracle, problems, paths, max_len, query, edits, sizes, ragged):
    postings = query + 1 if edits else 1
    buckets = 4
    while buckets * 8 < paths * max_len * postings:
        buckets *= 2
    filed = paths * sizes[0] * postings
    assert 8 * filed >= 5 * buckets and (problems - 8) * filed >= (64 if edits else 96) * buckets
    _appends(oracle, problems, paths, max_len, 40, query, edits, binding.MATCH_INDEX, sizes, ragged, few=3)


# what sorts its postings by bins of buckets first: paths around a sorting workgroup's 1024 positions, one
# and several problems, an empty index and one that holds postings, grams of up to four tokens and longer
# ones, few symbols (chains of many buckets, which lead through other bins).  (the assertion repeats the
# library's rule)
@pytest.mark.parametrize("problems,paths,max_len,vocab,query,edits,sizes", [
    (1, 64, 8300, 40, 3, 0, (8193, 3)),
    (1, 130, 4150, 6, 4, 0, (5, 4096)),
    (3, 50, 4200, 300, 6, 0, (70, 4097)),
    (1, 30, 3600, 40, 4, 1, (3500, 1, 60)),
    (2, 24, 1750, 12, 6, 1, (63, 1650)),
])
def test_appends_sorted_by_bins(oracle, problems, paths, max_len, vocab, query, edits, sizes):
    postings = query + 1 if edits else 1
    buckets = 4
    while buckets * 8 < paths * max_len * postings:
        buckets *= 2
    filed = paths * max(sizes) * postings
    assert buckets >= 1 << 14 and problems * paths * max_len * postings <= 1 << 22 and problems <= 8    # 256 bins
    assert problems * filed >= 1 << 19 and filed >= 256 * (256 if edits else 768)
    _appends(oracle, problems, paths, max_len, vocab, query, edits, binding.MATCH_INDEX, sizes, False)


@pytest.mark.parametrize("problems,paths,max_len,vocab,query,edits,n", [
    (1, 32, 4300, 40, 4, 1, 3600),
    (3, 50, 4200, 300, 6, 0, 4097),
])
def test_a_sorted_append_as_without_the_room_for_it(oracle, monkeypatch, problems, paths, max_len, vocab, query, edits, n):
    """Paths of different lengths, some of which the append fills up: clipped, with the status bit, by postings
    sorted first and, in a workspace that ends before the room for them, by claims on memory.  An id outside
    the vocabulary raises its bit."""
    print("sorted and not", problems, paths, max_len, vocab, query, edits, n, flush=True)
    rng = np.random.default_rng(n)
    postings, L, dev = (query + 1 if edits else 1), 6, torch.device("cuda:0")
    up = lambda size: (size + 255) // 256 * 256
    sources, bins = paths * ((max_len + 1023) // 1024), 256
    room = (up(problems * sources * 1024 * postings * 8) + up(problems * bins * sources * 4) +
            up(problems * paths * max_len * postings * 4) + up((problems * bins * 2 + 1) * 4))
    whole = binding.workspace_bytes(binding.Config(problems, paths, max_len, vocab, query, L, 1.0, 0, binding.MATCH_INDEX, edits, 0))
    assert problems * paths * n * postings >= 1 << 19 and paths * n * postings >= bins * (256 if edits else 768)
    offered = 2 * (max_len - n)
    counts = rng.integers(0, offered + 1, size=(problems, paths)).astype(np.int32)
    counts[:, 0], counts[:, 1] = offered, 0
    past, part = (rng.integers(0, vocab, size=(problems, paths, k)).astype(np.int32) for k in (offered, n))
    lens = np.minimum(counts + n, max_len).astype(np.int32)
    tokens = np.zeros((problems, paths, max_len), dtype=np.int32)
    for p, i in np.ndindex(problems, paths):
        path = np.concatenate([past[p, i, :counts[p, i]], part[p, i]])[:max_len]
        tokens[p, i, :len(path)] = path
    want = oracle.draft_all(tokens, None, lens, query, L, 1.0, 0, eps=edits)
    put = lambda a: torch.from_numpy(a).to(dev)
    dumps = []
    for nbytes in (whole, whole - room, whole - 256):
        monkeypatch.setattr(binding, "workspace_bytes", lambda cfg: nbytes)
        ix = binding.Index(problems, paths, max_len, vocab, query, L, 1.0, 0, binding.MATCH_INDEX, device=dev, max_edits=edits)
        ix.append(put(past), None, put(counts), offered)
        ix.append(put(part))
        out = ix.draft(query, L)
        assert np.array_equal(out["tokens"].cpu().numpy(), want["draft"])
        assert np.array_equal(out["length"].cpu().numpy(), want["draft_len"])
        assert ix.status() == binding.STATUS_CAPACITY
        dumps.append(ix.dump_matches(query, cap=1 << 22))
        ix.reset()
        bad = part.copy()
        bad[-1, -1, n // 2] = vocab
        ix.append(put(bad))
        assert ix.status() == binding.STATUS_TOKEN_RANGE
    for other in dumps[1:]:
        assert np.array_equal(dumps[0][0], other[0]) and np.array_equal(dumps[0][1], other[1])


def test_appends_of_a_few_tokens_to_many_rows(oracle):
    """8192 rows, 50 to 63 tokens each: the claims look at the fill counts first; two symbols: at full ones."""
    for vocab, query in ((40, 3), (2, 5)):
        _appends(oracle, 2048, 4, 200, vocab, query, 0, binding.MATCH_INDEX, (50, 63, 60), False)


def _appends(oracle, problems, N, T, vocab, query, edits, flags, sizes, ragged, few=0):
    """few: every so many problems take an eighth of the counts only."""
    rng = np.random.default_rng(problems * 1000 + vocab + query + edits)
    L = 6
    tokens = rng.integers(0, vocab, size=(problems, N, T)).astype(np.int32)
    motif = rng.integers(0, vocab, size=(problems, 1, 60)).astype(np.int32)
    cells = T // 60 * 60
    shared = rng.random((problems, N, T // 60)) < 0.5          # segments that the paths have in common
    tokens[:, :, :cells] = np.where(np.repeat(shared, 60, axis=2), np.tile(motif, (1, 1, T // 60)), tokens[:, :, :cells])
    probs = rng.random(tokens.shape).astype(np.float32)
    dev = torch.device("cuda:0")
    ix = binding.Index(problems, N, T, vocab, query, L, 0.5, 0, flags, device=dev, max_edits=edits)
    at = np.zeros((problems, N), dtype=np.int64)
    for turn, n in enumerate(sizes):
        print("append", problems, N, T, vocab, query, edits, flags, n, ragged, flush=True)
        counts = rng.integers(0, n + 1, size=at.shape) if ragged else np.full(at.shape, n)
        if ragged and few:
            counts[::few] //= 8
        idx = np.minimum(at[..., None] + np.arange(n), T - 1)
        step = lambda a: torch.from_numpy(np.ascontiguousarray(np.take_along_axis(a, idx, axis=2))).to(dev)
        ix.append(step(tokens), None if turn % 2 else step(probs),
                  torch.from_numpy(counts.astype(np.int32)).to(dev) if ragged else None, n)
        if turn % 2:                                           # no probabilities: all 1
            ones = np.arange(T) - at[..., None]
            probs[(ones >= 0) & (ones < counts[..., None])] = 1.0
        at += counts
        lens = at.astype(np.int32)
        out = ix.draft(query, L)
        want = oracle.draft_all(tokens, probs, lens, query, L, 0.5, 0, eps=edits)
        assert np.array_equal(out["tokens"].cpu().numpy(), want["draft"])
        assert np.array_equal(out["length"].cpu().numpy(), want["draft_len"])
        assert np.array_equal(out["path_scores"].cpu().numpy(), want["path_scores"].astype(np.float32))
    je, off = ix.dump_matches(query, cap=1 << 24)
    for r in range(0, problems * N, 1 if problems == 1 else 7 if problems < 1000 else 97):
        p, i = divmod(r, N)
        assert np.array_equal(je[off[r]:off[r + 1]], oracle.matches(tokens[p], lens[p], i, query, eps=edits))
    assert ix.status() == 0


def test_an_append_that_does_not_fit_is_clipped(oracle):
    """Counts beyond max_len: clipped, with the status bit, by both kernels."""
    rng = np.random.default_rng(9)
    for problems in (1, 72):                                  # (a thread per position / a workgroup per problem)
        tokens = rng.integers(0, 30, size=(problems, 4, 200)).astype(np.int32)
        ix = binding.Index(problems, 4, 150, 30, 3, 4, flags=binding.MATCH_INDEX)
        dev = torch.device("cuda:0")
        counts = torch.full((problems, 4), 90, dtype=torch.int32, device=dev)
        for first in (0, 90):
            part = np.ascontiguousarray(tokens[:, :, first:first + 100])
            ix.append(torch.from_numpy(part).to(dev), None, counts, 100)
        assert ix.status() == binding.STATUS_CAPACITY
        out = ix.draft(3, 4)
        want = oracle.draft_all(np.ascontiguousarray(tokens[:, :, :150]), None,
                                np.full((problems, 4), 150, dtype=np.int32), 3, 4, 1.0, 0)
        assert np.array_equal(out["tokens"].cpu().numpy(), want["draft"])


# a gram's sequence of buckets: more postings of one gram than its home block holds (all tokens the same: its chain
# goes through all blocks, and by the home block once more), filed posting by posting, by a workgroup per problem, by
# bins and by single steps, in tables of one block, of a few and of many
@pytest.mark.parametrize("problems,paths,max_len,query,edits,run,n", [
    (1, 8, 1024, 3, 0, 1.0, 1000),
    (1, 5, 60, 2, 0, 1.0, 50),
    (1, 4, 300, 3, 1, 1.0, 280),
    (12, 8, 300, 4, 0, 0.5, 290),
    (40, 6, 500, 3, 0, 0.7, 480),
    (1, 64, 4096, 4, 0, 0.02, 4000),
    (1, 64, 2048, 4, 1, 0.03, 2000),
])
def test_grams_that_fill_their_home_block(problems, paths, max_len, query, edits, run, n):
    print("home block", problems, paths, max_len, query, edits, run, flush=True)
    rng = np.random.default_rng(paths + n)
    tokens = rng.integers(1, 5000, size=(problems, paths, max_len)).astype(np.int32)
    same = rng.random((problems, paths, max_len // 20 + 1)) < run                  # runs of twenty of one token
    tokens = np.where(np.repeat(same, 20, axis=2)[:, :, :max_len], 7, tokens)
    tokens[:, :, n - 12:] = 7                                                      # ... which every path ends with
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a).astype(np.int32)).to("cuda:0")
    got = []
    for flags in (binding.MATCH_INDEX, binding.MATCH_SCAN):
        ix = binding.Index(problems, paths, max_len, 5000, query, 8, 1.0, 0, flags, device="cuda:0", max_edits=edits)
        ix.append(put(tokens[:, :, :n - 8]))
        for t in range(n - 8, n):
            ix.step(put(tokens[:, :, t]), None, None, 1, query, 8)
        got.append((ix.dump_matches(query, cap=1 << 24), ix.draft(query, 8), ix.status()))
    (matches, draft, status), (matches1, draft1, status1) = got
    assert np.array_equal(matches[1], matches1[1]) and np.array_equal(matches[0], matches1[0])
    for key in ("tokens", "length", "token_scores", "path_scores"):
        assert torch.equal(draft[key], draft1[key]), key
    assert status == status1 == 0 and int(matches[1][-1]) > 100


# a row whose matches lie far along a gram's sequence, behind the near part of a full home block where the index has such
# (from 2^17 positions): its own path, which it passes over, has that gram hundreds of times.  A row's step with its first
# four buckets at once, thousands of rows (a bucket first), one edit
@pytest.mark.parametrize("problems,paths,max_len,query,edits,blocks", [
    (1, 8, 800, 3, 0, False),
    (2, 40, 700, 6, 0, False),
    (300, 8, 700, 3, 0, False),
    (300, 7, 1300, 5, 0, False),
    (2, 8, 800, 3, 1, False),
    (1, 64, 4096, 3, 0, True),
    (1, 33, 6500, 5, 0, True),
    (16, 128, 2048, 4, 0, True),
    (1, 64, 2048, 3, 1, True),
])
def test_steps_whose_matches_lie_far_along_a_sequence(problems, paths, max_len, query, edits, blocks):
    print("far along", problems, paths, max_len, query, edits, flush=True)
    assert blocks == (paths * max_len > 1 << 17 or (edits > 0 and paths * max_len * (query + 1) >= 1 << 19))
    rng = np.random.default_rng(problems + paths)
    n, n_steps = max_len - 40, 4
    tokens = rng.integers(10, 5000, size=(problems, paths, max_len)).astype(np.int32)
    tokens[:, 0] = 7                                                       # n postings of it, 15 to a bucket
    for at in range(n - 60, n - 20, 20):
        tokens[:, 1:, at:at + query + 1] = 7                               # ... and a few with other tokens behind
        tokens[:, 1:, at + query + 1:at + query + 4] = rng.integers(10, 14, size=(problems, paths - 1, 3))
    tokens[:, 1::2, n:n + n_steps] = 7
    assert (n - 60) > 15 * 32 + query
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a).astype(np.int32)).to("cuda:0")
    outs = []
    for flags in (binding.MATCH_INDEX, binding.MATCH_SCAN):
        ix = binding.Index(problems, paths, max_len, 5000, query, 8, 1.0, 0, flags, device="cuda:0", max_edits=edits)
        ix.append(put(tokens[:, :1, :n].repeat(paths, axis=1)), None,
                  put(np.where(np.arange(paths) == 0, n - 60, 0)[None].repeat(problems, axis=0)))
        ix.append(put(tokens[:, :, :n]), None, put(np.where(np.arange(paths) == 0, 0, n)[None].repeat(problems, axis=0)))
        outs.append([ix.step(put(tokens[:, :, t]), None, None, 1, query, 8) for t in range(n, n + n_steps)] + [ix.draft(query, 8)])
        assert ix.status() == 0
    for a, b in zip(*outs):
        for key in ("tokens", "length", "token_scores", "path_scores"):
            assert torch.equal(a[key], b[key]), key
    assert int(outs[0][0]["length"][:, 0].min()) > 0 and int(outs[0][0]["tokens"][:, 0].max()) >= 10


# indexes with home blocks under the other kernels that file and look up: replays by lanes (2^15 drafts), the accept-driven
# loop in one launch, and all steps of either by a workgroup per problem
@pytest.mark.parametrize("problems,paths,max_len,query,steps", [(8, 64, 4096, 3, 64), (1, 16, 16000, 3, 40), (2, 12, 15000, 4, 30), (1, 6, 40000, 3, 30)])
def test_home_blocks_under_replays_and_loops(problems, paths, max_len, query, steps):
    print("home blocks", problems, paths, max_len, query, steps, flush=True)
    assert paths * max_len > 1 << 17
    rng = np.random.default_rng(paths)
    tokens = rng.integers(1, 40000, size=(problems, paths, max_len)).astype(np.int32)
    same = rng.random((problems, paths, max_len // 20 + 1)) < 0.004                # runs of twenty of one token, and
    tokens = np.where(np.repeat(same, 20, axis=2)[:, :, :max_len], 7, tokens)
    shared = rng.random((problems, paths, max_len // 20 + 1)) < 0.4                # ... of one path's earlier ones
    tokens = np.where(np.repeat(shared, 20, axis=2)[:, :, :max_len], np.roll(tokens[:, :1], 60, axis=2), tokens).astype(np.int32)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    n = max_len - steps
    futures, now, past = put(tokens), put(tokens[:, :, n:].transpose(2, 0, 1)), put(tokens[:, :, :n])
    outs = []
    for per_launch in (1, 0, 1 << 20):
        if per_launch > 1 and paths > 16:
            continue
        ix = binding.Index(problems, paths, max_len, 40000, query, 8, 0.5, 0, binding.MATCH_INDEX, device="cuda:0")
        if per_launch:
            ix.set_steps_per_launch(per_launch)
        ix.append(past)
        got = [ix.replay(steps, now, None, query, 8)]
        if paths <= 16:
            ix.reset()
            ix.append(past)
            got.append(ix.accept_loop(steps // 5, futures, None, query, 8))
        outs.append((got + [ix.draft(query, 8)], ix.status()))
    for got, status in outs[1:]:
        assert status == outs[0][1]
        for a, b in zip(outs[0][0], got):
            for key in ("tokens", "length", "token_scores", "path_scores", "accept", "path_len"):
                if a.get(key) is not None and b.get(key) is not None:
                    assert torch.equal(a[key], b[key]), key
    assert int(outs[0][0][0]["length"].sum()) > 0


@pytest.mark.parametrize("problems,paths,max_len,query", [(20, 16, 2048, 3), (19, 8, 4096, 5)])
def test_a_workgroup_per_problem_in_an_index_with_home_blocks(problems, paths, max_len, query):
    """One edit: histories as a whole are sorted, with counts each problem is filed by a workgroup, from
    behind what is there; a frequent gram fills its home block."""
    print("home blocks, counts", problems, paths, max_len, query, flush=True)
    rng = np.random.default_rng(problems)
    tokens = rng.integers(1, 5000, size=(problems, paths, max_len)).astype(np.int32)
    runs = rng.random((problems, paths, max_len // 20 + 1)) < 0.04
    tokens = np.where(np.repeat(runs, 20, axis=2)[:, :, :max_len], 7, tokens).astype(np.int32)
    tokens[:, 1:, -200:-40] = tokens[:, :1, -500:-340]
    tokens[:, 0, -60:-40] = tokens[:, 0, -500:-480]
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    n, first = max_len - 40, 30
    counts = np.full((problems, paths), n - first, dtype=np.int32)
    counts[:, 1::3] -= 17
    outs = []
    for flags, sort in ((binding.MATCH_INDEX, False), (binding.MATCH_INDEX, True), (binding.MATCH_SCAN, False)):
        ix = binding.Index(problems, paths, max_len, 5000, query, 8, 1.0, 0, flags, device="cuda:0", max_edits=1)
        if sort:                                           # the same histories, without counts
            ix.append(put(tokens[:, :, :n - 17]))
            more = np.zeros_like(counts)
            more[counts == n - first] = 17
            ix.append(put(tokens[:, :, n - 17:n]), None, put(more))
        else:
            ix.append(put(tokens[:, :, :first]))
            ix.append(put(tokens[:, :, first:n]), None, put(counts))
        outs.append((ix.draft(query, 8), ix.dump_matches(query, cap=1 << 22), ix.status()))
    for out, matches, status in outs[:2]:
        for key in ("tokens", "length", "token_scores", "path_scores"):
            assert torch.equal(out[key], outs[2][0][key]), key
        assert np.array_equal(matches[0], outs[2][1][0]) and np.array_equal(matches[1], outs[2][1][1]) and status == 0
    assert int(outs[0][0]["length"].sum()) > 0

"""csd_replay with its steps side by side against a launch per step (csd_set_steps_per_launch 1; other
tests compare both with the oracle): every output, the index left behind, status bits."""
import numpy as np
import pytest
import torch

from paper_2503_05330_amd import binding

pytestmark = pytest.mark.gpu

KEYS = ("tokens", "length", "token_scores", "path_scores", "accept")


def _same(a, b):
    for key in KEYS:
        x, y = a[key].cpu().numpy(), b[key].cpu().numpy()
        assert np.array_equal(x.view(np.int32), y.view(np.int32)), key


# paths around the 16 of a workgroup and a wave; steps around a workgroup's threads; several launches
# (a quarter of max_len steps each); options, pools and matchers; one and several problems
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,edits,flags,pool", [
    (1, 16, 300, 3, 3, 8, 0, binding.MATCH_AUTO, 0),
    (1, 17, 200, 65, 4, 10, 0, binding.MATCH_AUTO, 0),
    (1, 1, 90, 70, 2, 4, 0, binding.MATCH_AUTO | binding.INCLUDE_SELF, 0),
    (3, 5, 1300, 1100, 3, 8, 0, binding.MATCH_AUTO, 0),
    (1, 66, 150, 64, 6, 32, 0, binding.MATCH_AUTO, 0),
    (7, 64, 130, 33, 2, 16, 0, binding.MATCH_AUTO, 0),
    (300, 30, 128, 66, 3, 8, 0, binding.MATCH_AUTO, 0),
    (2, 9, 200, 40, 3, 6, 0, binding.MATCH_SCAN, 0),
    (1, 16, 300, 32, 3, 8, 1, binding.MATCH_AUTO, 0),
    (2, 20, 300, 31, 4, 10, 1, binding.MATCH_INDEX, 0),
    (1, 6, 120, 50, 5, 17, 1, binding.MATCH_INDEX, 0),
    (1, 5, 100, 20, 3, 5, 2, binding.MATCH_AUTO, 0),
    (2, 13, 200, 30, 3, 7, 0, binding.MATCH_AUTO, 1),
    (2, 13, 200, 31, 3, 7, 1, binding.MATCH_AUTO, 2),
    (1, 8, 150, 30, 4, 6, 0, binding.MATCH_AUTO | binding.QUERY_BACKOFF, 0),
    (1, 8, 150, 30, 4, 6, 0, binding.MATCH_INDEX | binding.QUERY_BACKOFF | binding.INCLUDE_SELF, 2),
])
@pytest.mark.parametrize("start", ("empty", "ragged", "full"))
def test_steps_side_by_side(problems, paths, max_len, steps, query, draft, edits, flags, pool, start):
    rng = np.random.default_rng(problems * 100 + paths + steps + query)
    print("replay", problems, paths, max_len, steps, query, draft, edits, flags, pool, start, flush=True)
    dev, V, T = torch.device("cuda:0"), 60, max_len
    tokens = rng.integers(0, V, size=(problems, paths, T)).astype(np.int32)
    motif = np.tile(rng.integers(0, V, size=(problems, 1, 50)).astype(np.int32), (1, 1, T // 50 + 1))[:, :, :T]
    tokens = np.where(np.repeat(rng.random((problems, paths, T // 10 + 1)) < 0.5, 10, axis=2)[:, :, :T], motif, tokens)
    probs = rng.random(tokens.shape).astype(np.float32)
    counts = {"empty": np.zeros((problems, paths)), "ragged": rng.integers(0, T - steps, size=(problems, paths)),
              # some paths full before the first step, some during the replay
              "full": rng.integers(max(0, T - 2 * steps), T + 1, size=(problems, paths))}[start].astype(np.int32)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    later = (T // 3 + np.arange(steps + 1)) % T
    d_tok, d_probs = put(tokens[:, :, later].transpose(2, 0, 1)), put(probs[:, :, later].transpose(2, 0, 1))
    targets = rng.integers(0, V, size=(steps, problems, paths, draft)).astype(np.int32)
    got = []
    for per_launch in (0, 1):
        ix = binding.Index(problems, paths, T, V, query, draft, 0.6, 0, flags, device=dev, max_edits=edits, pool_mode=pool)
        if start != "empty":                              # (counts: the library does not know the lengths)
            ix.append(put(tokens), put(probs), put(counts), T)
        if per_launch:
            ix.set_steps_per_launch(per_launch)
        use_probs = d_probs[:steps].contiguous() if steps % 2 else None
        out = ix.replay(steps, d_tok[:steps], use_probs, query, draft, targets=put(targets))
        # the length of the drafts that the index now holds the basis for, and one step more
        after = ix.draft(query, draft)
        more = ix.step(d_tok[steps], None, torch.ones((problems, paths), dtype=torch.int32, device=dev), 1, query, draft)
        got.append((out, after, more, ix.dump_matches(query, cap=1 << 23) if problems * paths < 500 else None, ix.status()))
    (a, b, c, d, e), (a1, b1, c1, d1, e1) = got
    _same(a, a1)
    for x, y in ((b, b1), (c, c1)):
        for key in KEYS[:4]:
            assert torch.equal(x[key], y[key]), key
    if d is not None:
        assert np.array_equal(d[0], d1[0]) and np.array_equal(d[1], d1[1])
    assert e == e1 and (e == 0 or start == "full")
    assert int(a["length"].sum()) > 0 or start == "empty"


# enough drafts for the kernels with four and eight lanes per draft, which small problems take where it does not pay to hand
# a CU to each: drafts of one to 30 tokens, grams of two to six, rows with no, few, many and hundreds of matches (two
# symbols: chains of full buckets), edge scoring, more than 64 paths, short paths, a wave's sixteen rows across problems
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,mode,warm", [
    (64, 16, 200, 40, 3, 8, 60, 0, 150),
    (64, 17, 160, 31, 4, 13, 60, 1, 120),
    (3, 70, 640, 160, 6, 30, 40, 0, 90),
    (1, 64, 2100, 520, 5, 16, 2000, 0, 150),
    (1100, 5, 60, 7, 2, 5, 2, 1, 40),
    (2100, 2, 64, 8, 1, 1, 300, 0, 50),
    (130, 16, 100, 20, 3, 7, 9, 0, 0),
])
def test_many_drafts_side_by_side(problems, paths, max_len, steps, query, draft, vocab, mode, warm):
    _many(problems, paths, max_len, steps, query, query, draft, vocab, mode, warm)


# the same with problems larger than a workgroup's LDS (2^14 positions), which all take those kernels: the usual grams and
# drafts, both weights, an eighth's rows pooled by four and by sixteen waves (2^17 drafts), rows left over or none
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,mode,warm", [
    (32, 20, 1024, 64, 3, 8, 3000, 0, 900),
    (32, 20, 1024, 64, 3, 8, 60, 1, 900),
    (64, 40, 512, 64, 4, 13, 2000, 1, 400),
    (130, 33, 500, 31, 4, 8, 500, 0, 300),
    (16, 70, 250, 40, 2, 5, 6, 1, 200),
])
def test_many_drafts_of_large_problems(problems, paths, max_len, steps, query, draft, vocab, mode, warm):
    assert paths * ((max_len + 3) // 4 * 4) > 1 << 14
    _many(problems, paths, max_len, steps, query, query, draft, vocab, mode, warm)


def test_many_drafts_of_a_shorter_query():
    """Queries shorter than the index's grams are scanned for: a wave per draft, however many there are."""
    _many(64, 16, 200, 40, 4, 2, 8, 60, 0, 150)
    _many(64, 16, 200, 40, 6, 5, 12, 30, 1, 150)


def _many(problems, paths, max_len, steps, longest, query, draft, vocab, mode, warm):
    rng = np.random.default_rng(problems + paths + vocab)
    print("many", problems, paths, max_len, steps, query, draft, vocab, mode, warm, flush=True)
    dev, T = torch.device("cuda:0"), max_len
    assert problems * paths * steps >= 1 << 15 and steps <= max(T // 4, 16)     # in one launch
    tokens = rng.integers(0, vocab, size=(problems, paths, T)).astype(np.int32)
    pool = rng.integers(0, vocab, size=(problems, 1, 12, 10)).astype(np.int32)      # segments in any order
    order = rng.integers(0, 12, size=(problems, paths, T // 10 + 1))
    shared = np.take_along_axis(np.repeat(pool, paths, axis=1), order[..., None], axis=2).reshape(problems, paths, -1)[:, :, :T]
    tokens = np.where(rng.random(tokens.shape) < 0.9, shared, tokens)
    # (few distinct probabilities: equal weights, decided by the lower token)
    probs = (rng.integers(0, 5, size=tokens.shape) / 4.0).astype(np.float32)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    targets = put(np.concatenate([tokens, tokens], 2)[:, :, warm + 1:warm + 1 + steps + draft].astype(np.int32))
    targets = targets.unfold(2, draft, 1)[:, :, :steps].permute(2, 0, 1, 3).contiguous()
    by_step = lambda a: put(a[:, :, warm:warm + steps].transpose(2, 0, 1))
    got = []
    for per_launch in (0, 1):
        ix = binding.Index(problems, paths, T, vocab, longest, draft, 0.7, mode, binding.MATCH_INDEX, device=dev)
        if warm:
            counts = np.where(np.arange(paths) % 5 == 4, warm // 3, warm) + np.zeros((problems, 1))
            ix.append(put(tokens[:, :, :warm]), put(probs[:, :, :warm]), put(counts.astype(np.int32)), warm)
        if per_launch:
            ix.set_steps_per_launch(per_launch)
        got.append((ix.replay(steps, by_step(tokens), by_step(probs), query, draft, targets=targets), ix.status()))
    (a, status), (b, status1) = got
    _same(a, b)
    assert status == status1 == 0
    assert int(a["length"].sum()) > 0 and int(a["accept"].sum()) > 0


def test_a_captured_replay_goes_on_from_where_it_was():
    """An even number of steps leaves the paths' ends where it found them: a captured replay, run
    again and again with other work between, appends again each time."""
    rng = np.random.default_rng(3)
    dev, P, N, T, V, S, k, L = torch.device("cuda:0"), 2, 6, 400, 30, 8, 3, 8
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    tokens = rng.integers(0, V, size=(5, S, P, N)).astype(np.int32)
    past = put(rng.integers(0, V, size=(P, N, 300)).astype(np.int32))
    by_graph, by_call = (binding.Index(P, N, T, V, k, L, device=dev) for _ in range(2))
    by_call.set_steps_per_launch(1)
    fed = put(tokens[0])
    out = by_graph._outputs(L, True, lead=(S,))
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        by_graph.append(past)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            by_graph.replay(S, fed, None, k, L, out=out)
    by_call.append(past)
    for turn in range(5):
        fed.copy_(put(tokens[turn]))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = by_call.replay(S, put(tokens[turn]), None, k, L)
        for key in KEYS[:4]:
            assert torch.equal(out[key], want[key]), (turn, key)


# (a wave per draft; a workgroup per problem, its histories in LDS; four lanes a draft, problems of more than 2^14 positions)
@pytest.mark.parametrize("problems,paths,steps", [(1, 6, 20), (64, 32, 17), (64, 48, 17)])
def test_a_step_fed_with_what_an_earlier_one_drafted(problems, paths, steps):
    """Drafts of one token written where the next step's tokens are read from: the steps see each
    other's drafts, as they do in a launch per step."""
    print("fed", problems, paths, steps, flush=True)
    dev, V, k, warm = torch.device("cuda:0"), 40, 3, 60
    start = np.random.default_rng(steps).integers(0, 7, size=(problems, paths, 1))
    past = ((start + np.arange(warm)) % 13).astype(np.int32)     # the same cycle from different places on
    cells = torch.full((steps + 1, problems, paths), 39, dtype=torch.int32, device=dev)
    cells[0] = torch.from_numpy((past[:, :, -1] + 1) % 13).to(dev)
    out = dict(tokens=cells[1:], length=torch.empty((steps, problems, paths), dtype=torch.int32, device=dev))
    ix = binding.Index(problems, paths, 400, V, k, 1, device=dev)
    ix.append(torch.from_numpy(past).to(dev))
    assert problems == 1 or problems * paths * steps >= 1 << 15    # all forms of a replay side by side
    ix.replay(steps, cells[:-1], None, k, 1, out=out, scores=False)
    want = (past[None, :, :, -1] + 1 + np.arange(steps + 1)[:, None, None]) % 13
    assert np.array_equal(cells.cpu().numpy(), want)
    assert ix.status() == 0


@pytest.mark.parametrize("problems,paths,steps", [(1, 6, 20), (64, 32, 17), (64, 96, 17)])
def test_accepted_lengths_in_the_place_of_the_drafts(problems, paths, steps):
    """One buffer for both: it holds the accepted lengths, which are written last."""
    rng = np.random.default_rng(steps + 1)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    V, k, L, S = (6 if problems == 1 else 40), 2, 4, steps  # (rows with few matches)
    tokens, targets = (rng.integers(0, V, size=s).astype(np.int32) for s in ((S, problems, paths), (S, problems, paths, L)))
    past = rng.integers(0, V, size=(problems, paths, 100)).astype(np.int32)
    accepted = []
    for shared in (False, True):
        ix = binding.Index(problems, paths, 200, V, k, L, device="cuda:0")
        ix.append(put(past))
        out = ix._outputs(L, True, lead=(S,))
        where = out["length"] if shared else torch.empty_like(out["length"])
        ix.replay(S, put(tokens), None, k, L, out=out, targets=put(targets), accept_out=where)
        accepted.append(where)
    assert torch.equal(*accepted) and int(accepted[0].sum()) > 0


@pytest.mark.parametrize("edits,flags", [(0, binding.MATCH_INDEX), (1, binding.MATCH_INDEX), (1, binding.MATCH_SCAN)])
def test_a_workspace_without_the_part_for_speed(monkeypatch, edits, flags):
    """The size that histories, ends, index and shared scans take is enough; a byte less is not."""
    P, N, T, V, k, L, S = 2, 5, 900, 20, 3, 6, 30
    up = lambda n: (n + 255) // 256 * 256
    indexed = flags == binding.MATCH_INDEX
    stride = (1 + k + (1 if indexed and edits else 0) + 3) // 4 * 4
    size = 2 * up((P * N * T + 32) * 4) + 2 * up(P * N * stride * 4) + up(16)
    if indexed:
        buckets = 4
        while buckets * 8 < N * T * (k + 1 if edits else 1):
            buckets *= 2
        size += up(P * buckets * 64)
    else:                                                  # a list of 4096 matches and a state word a path
        size += up(P * N * 4096 * 8) + up(P * N * 8)
    rng = np.random.default_rng(2)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    past, more, tokens = (put(rng.integers(0, V, size=s).astype(np.int32)) for s in ((P, N, 600), (P, N, 70), (S, P, N)))
    make = lambda: binding.Index(P, N, T, V, k, L, 1.0, 0, flags, device="cuda:0", max_edits=edits)
    got = []
    full = binding.workspace_bytes(binding.Config(P, N, T, V, k, L, 1.0, 0, flags, edits, 0))
    for nbytes in (full, size):
        monkeypatch.setattr(binding, "workspace_bytes", lambda cfg: nbytes)
        ix = make()
        ix.append(past)
        ix.append(more)
        got.append(ix.replay(S, tokens, None, k, L, targets=torch.zeros((S, P, N, L), dtype=torch.int32, device="cuda:0")))
        assert ix.status() == 0
    _same(*got)
    assert int(got[0]["length"].sum()) > 0 and size < full
    monkeypatch.setattr(binding, "workspace_bytes", lambda cfg: size - 1)
    with pytest.raises(binding.CsdError):
        make()


# the scan, one row a CU, its candidates pooled by wave: paths around a span of 256 positions and the
# first positions of a path, large problems; symbols few enough for rows of up to a wave's, a workgroup's
# and the match list's worth of matches and beyond
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,edits,mode", [
    (1, 2, 9, 6, 3, 4, 4, 1, 0),
    (2, 5, 255, 5, 3, 8, 30, 1, 0),
    (1, 3, 257, 5, 2, 3, 9, 1, 1),
    (3, 16, 258, 4, 4, 8, 12, 1, 0),
    (1, 16, 1024, 3, 3, 8, 40, 1, 0),
    (1, 32, 2048, 2, 3, 8, 150, 1, 0),
    (1, 16, 1024, 2, 3, 32, 12, 1, 0),
    (1, 9, 700, 3, 4, 16, 20, 1, 1),
    (1, 9, 700, 3, 3, 6, 6, 0, 0),
    (1, 8, 400, 2, 4, 5, 5, 2, 0),
    (1, 33, 2048, 2, 3, 8, 150, 1, 0),
    (1, 9, 700, 3, 6, 8, 8, 1, 0),
])
def test_scanned_rows_beside_each_other(oracle, problems, paths, max_len, steps, query, draft, vocab, edits, mode):
    _against_the_oracle(oracle, problems, paths, max_len, steps, query, draft, vocab, edits, mode, binding.MATCH_SCAN)


# the same with two rows a CU, which takes more drafts: fewest of them, largest problems by the tokens that
# an edit leaves of the query.  (the assertion repeats the library's rule)
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,edits,mode", [
    (48, 2, 9, 6, 3, 4, 4, 1, 0),
    (20, 5, 255, 6, 3, 8, 30, 1, 0),
    (35, 3, 257, 5, 2, 3, 9, 1, 1),
    (8, 16, 258, 4, 4, 8, 12, 1, 0),
    (1, 16, 1024, 32, 3, 8, 40, 1, 0),
    (1, 32, 2048, 16, 4, 8, 60, 1, 0),
    (2, 16, 512, 16, 2, 32, 8, 1, 0),
    (1, 16, 1024, 32, 3, 32, 12, 1, 0),
    (10, 9, 700, 6, 4, 16, 20, 1, 1),
    (7, 9, 700, 5, 3, 6, 6, 0, 0),
    (1, 32, 2048, 9, 3, 8, 40, 0, 0),
    (13, 8, 400, 5, 4, 5, 5, 2, 0),
    (16, 4, 1024, 8, 1, 8, 5, 0, 0),
])
def test_scanned_rows_two_a_cu(oracle, problems, paths, max_len, steps, query, draft, vocab, edits, mode):
    left = query - edits
    assert paths * max_len <= 1 << (16 if left >= 3 else 14 if left == 2 else 13 if edits else 12)
    assert problems * paths * steps >= (512 if edits or left < 2 else 257)
    _against_the_oracle(oracle, problems, paths, max_len, steps, query, draft, vocab, edits, mode, binding.MATCH_SCAN)


# one edit through the index with more drafts than are under way at once: rows of up to 64 matches, of a
# workgroup's worth and of more (few symbols), drafts whose windows hold fewer matches than a wave has
# lanes, chains of many buckets and queries of up to eight tokens, paths shorter than a gram, all pools
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,mode,pool", [
    (1, 16, 256, 40, 4, 8, 12, 0, 0),
    (2, 9, 300, 30, 4, 16, 9, 1, 0),
    (3, 20, 100, 10, 2, 4, 14, 0, 0),
    (1, 66, 130, 8, 5, 32, 7, 0, 0),
    (1, 26, 120, 20, 8, 10, 3, 0, 0),
    (1, 30, 400, 18, 3, 8, 5, 1, 0),
    (1, 70, 200, 8, 4, 8, 4, 0, 0),
    (60, 3, 12, 3, 4, 5, 3, 0, 0),
    (1, 20, 300, 26, 4, 7, 10, 0, 1),
    (1, 40, 260, 13, 3, 6, 6, 0, 2),
])
def test_rows_left_to_workgroups(oracle, problems, paths, max_len, steps, query, draft, vocab, mode, pool):
    assert problems * paths * steps > 512 and steps <= max(max_len // 4, 16)
    _against_the_oracle(oracle, problems, paths, max_len, steps, query, draft, vocab, 1, mode, binding.MATCH_INDEX, pool)


# the same with a path's own history and with queries that lose tokens until they match (symbols enough for
# rows without a match), in the launch of the waves and in that of the workgroups
@pytest.mark.parametrize("flags", (binding.INCLUDE_SELF, binding.QUERY_BACKOFF, binding.INCLUDE_SELF | binding.QUERY_BACKOFF))
@pytest.mark.parametrize("problems,paths,max_len,steps,query,draft,vocab,mode,pool", [
    (1, 16, 256, 40, 4, 8, 12, 0, 0),
    (2, 9, 300, 30, 4, 16, 60, 1, 0),
    (40, 4, 60, 4, 5, 6, 90, 0, 1),
    (1, 40, 260, 13, 3, 6, 6, 0, 2),
])
def test_rows_left_to_workgroups_with_options(oracle, problems, paths, max_len, steps, query, draft, vocab, mode, pool, flags):
    assert problems * paths * steps > 512 and steps <= max(max_len // 4, 16)
    _against_the_oracle(oracle, problems, paths, max_len, steps, query, draft, vocab, 1, mode, binding.MATCH_INDEX, pool, flags)


def _against_the_oracle(oracle, problems, paths, max_len, steps, query, draft, vocab, edits, mode, matcher, pool=0, flags=0):
    rng = np.random.default_rng(paths * max_len + vocab)
    print("oracle", matcher, flags, pool, problems, paths, max_len, steps, query, draft, vocab, edits, mode, flush=True)
    dev, warm = torch.device("cuda:0"), max_len - steps
    tokens = rng.integers(0, vocab, size=(problems, paths, max_len)).astype(np.int32)
    motif = rng.integers(0, vocab, size=(problems, 1, max_len)).astype(np.int32)
    tokens = np.where(rng.random(tokens.shape) < 0.3, motif, tokens)
    probs = rng.random(tokens.shape).astype(np.float32)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ix = binding.Index(problems, paths, max_len, vocab, query, draft, 0.7, mode, matcher | flags, device=dev, max_edits=edits,
                       pool_mode=pool)
    counts = rng.integers(warm // 2, warm + 1, size=(problems, paths)).astype(np.int32)
    counts[:, 0] = warm
    ix.append(put(tokens[:, :, :warm]), put(probs[:, :, :warm]), put(counts), warm)
    later = np.take_along_axis(tokens, np.minimum(counts[..., None] + np.arange(steps), max_len - 1), axis=2)
    later_probs = np.take_along_axis(probs, np.minimum(counts[..., None] + np.arange(steps), max_len - 1), axis=2)
    out = ix.replay(steps, put(later.transpose(2, 0, 1)), put(later_probs.transpose(2, 0, 1)), query, draft)
    lengths = (counts[None] + np.arange(1, steps + 1)[:, None, None]).astype(np.int32)
    want = oracle.draft_many(tokens, probs, lengths, query, draft, 0.7, mode, eps=edits, pool_mode=pool,
                             include_self=bool(flags & binding.INCLUDE_SELF), backoff=bool(flags & binding.QUERY_BACKOFF))
    for key, name in (("tokens", "draft"), ("length", "draft_len"), ("token_scores", "token_scores"), ("path_scores", "path_scores")):
        assert np.array_equal(out[key].cpu().numpy().view(np.int32), want[name].view(np.int32)), key
    assert ix.status() == 0

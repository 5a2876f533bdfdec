"""Calls that append, captured in a HIP graph: every replay goes on from where the paths are, also with
eager calls on the same handle in between, as the same calls made one by one do (which other tests
compare with the oracle)."""
import numpy as np
import pytest
import torch

from paper_2503_05330_amd import binding

pytestmark = pytest.mark.gpu

KEYS = ("tokens", "length", "token_scores", "path_scores")


def _put(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _tokens(rng, problems, paths, n, vocab):
    """Histories with segments in common."""
    motif = np.tile(rng.integers(0, vocab, size=(problems, 1, 40)), (1, 1, n // 40 + 1))[:, :, :n]
    shared = np.repeat(rng.random((problems, paths, n // 20 + 1)) < 0.6, 20, axis=2)[:, :, :n]
    return np.where(shared, motif, rng.integers(0, vocab, size=(problems, paths, n))).astype(np.int32)


def _same(got, want, keys=KEYS):
    for key in keys:
        assert torch.equal(got[key], want[key]), key


def _captured(call):
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        kept = call()
    return graph, kept


# a workgroup for a path's tokens and several of them; a workgroup per problem (many problems, a good
# part of their indexes at once); postings sorted first; matching by scan; a step that appends first (many tokens, or one-edit
# matching); the ends of an odd number of appends
@pytest.mark.parametrize("problems,paths,max_len,query,edits,flags,call,n", [
    (1, 4, 4000, 3, 0, binding.MATCH_INDEX, "append", 1),
    (1, 4, 4000, 3, 0, binding.MATCH_INDEX, "append", 600),
    (2, 3, 2000, 6, 0, binding.MATCH_INDEX, "append", 257),
    (1, 4, 2000, 3, 1, binding.MATCH_INDEX, "append", 300),
    (1, 4, 2000, 3, 0, binding.MATCH_SCAN, "append", 300),
    (1, 4, 700, 3, 1, binding.MATCH_SCAN, "append", 65),
    (64, 5, 300, 3, 0, binding.MATCH_INDEX, "append", 90),
    (64, 20, 1000, 3, 0, binding.MATCH_INDEX, "append", 352),
    (40, 5, 720, 3, 1, binding.MATCH_INDEX, "append", 210),
    (1, 32, 8300, 3, 1, binding.MATCH_INDEX, "append", 4097),
    (1, 4, 900, 3, 0, binding.MATCH_INDEX, "step", 70),
    (2, 5, 400, 3, 1, binding.MATCH_INDEX, "step", 3),
    (112, 5, 720, 3, 0, binding.MATCH_INDEX, "step", 100),
    (2, 5, 400, 3, 0, binding.MATCH_INDEX, "replay", 3),
    (2, 5, 400, 3, 1, binding.MATCH_SCAN, "replay", 3),
    (2, 5, 400, 5, 0, binding.MATCH_INDEX, "loop", 3),
    (2, 5, 400, 3, 1, binding.MATCH_INDEX, "loop", 3),
    # all steps in one launch, with the minimum of scratch memory and with twice as much
    (2, 5, 400, 3, 0, binding.MATCH_INDEX, "loop", 3),
    (1, 16, 400, 4, 0, binding.MATCH_INDEX, "loop", 3),
    (1, 20, 400, 4, 0, binding.MATCH_INDEX, "loop", 3),
    (2, 5, 400, 3, 0, binding.MATCH_INDEX, "loop, twice the scratch", 3),
])
def test_a_captured_append_goes_on_from_where_it_was(problems, paths, max_len, query, edits, flags, call, n):
    print("captured", problems, paths, max_len, query, edits, flags, call, n, flush=True)
    rng = np.random.default_rng(problems + paths + max_len + n)
    L, V, warm = 6, (30 if n > 3 else 3), 20
    turns = min(5, (max_len - warm - 7) // n)
    fed_at = [_tokens(rng, problems, paths, n, V) for _ in range(turns)]
    if call == "replay":
        fed_at = [a.transpose(2, 0, 1) for a in fed_at]
    elif call.startswith("loop"):
        fed_at = [_tokens(rng, problems, paths, max_len, V)] * turns
    past, between = (_put(_tokens(rng, problems, paths, k, V)) for k in (warm, 7))
    by_graph, by_call = (binding.Index(problems, paths, max_len, V, query, L, 0.5, 0, flags, device="cuda:0", max_edits=edits)
                         for _ in range(2))
    fed = _put(fed_at[0])

    def go(ix, tokens, out):
        if call == "append":
            ix.append(tokens)
            out = ix.draft(query, L, out=out)
            out["accept"] = ix.accept(out["tokens"], out["length"], out["tokens"], L)
        elif call == "step":
            out = ix.step(tokens, None, None, n, query, L, out=out)
        elif call == "replay":
            out = ix.replay(n, tokens, None, query, L, out=out, fused=False)
        else:
            out = ix.accept_loop(n, tokens, None, query, L, min_scratch=call == "loop")
        return out
    for ix in (by_graph, by_call):
        ix.append(past)
    graph, out = _captured(lambda: go(by_graph, fed, None))
    keys = ("tokens", "length", "accept", "path_len") if call.startswith("loop") else KEYS
    drafted = 0
    for turn in range(turns):
        fed.copy_(_put(fed_at[turn]))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = go(by_call, _put(fed_at[turn]), None)
        _same(out, want, keys)
        drafted += int(want["length"].sum())
        if turn == 1:                                     # an eager call in between
            for ix in (by_graph, by_call):
                ix.append(between)
            _same(by_graph.draft(query, L), by_call.draft(query, L))
    a, b = (ix.dump_matches(query, cap=1 << 22) for ix in (by_graph, by_call))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert drafted > 0
    assert by_graph.status() == by_call.status() == 0


# the buckets of a problem in LDS, and their fill counts only; postings sorted first
@pytest.mark.parametrize("problems,paths,max_len,edits,n", [(64, 5, 300, 0, 100), (40, 6, 800, 1, 360), (1, 32, 8300, 1, 4097)])
def test_a_bulk_append_keeps_what_a_graph_has_appended(problems, paths, max_len, edits, n):
    """An index that no call has appended to since its reset is not empty if a graph has: a bulk append
    (by a workgroup per problem, or sorted by bins) keeps the graph's postings, captured or not."""
    print("bulk behind a graph", problems, paths, max_len, edits, n, flush=True)
    rng = np.random.default_rng(paths + n)
    P, L, V, k = problems, 6, 6, 3
    make = lambda: binding.Index(P, paths, max_len, V, k, L, 0.5, 0, binding.MATCH_INDEX, device="cuda:0", max_edits=edits)
    part = [_put(_tokens(rng, P, paths, n, V)) for _ in range(2)]
    want = make()
    for tokens in part:
        want.append(tokens)
    by_graph, mixed = make(), make()
    fed = part[0].clone()
    twice, _ = _captured(lambda: by_graph.append(fed))     # captured on an empty index, replayed twice
    small = part[0][:, :, :1].contiguous()                 # (an append too small for these forms)
    few, _ = _captured(lambda: mixed.append(small))
    mixed.reset()                                          # nothing of the capture has run: no call knows of the graph's tokens
    for tokens in part:
        fed.copy_(tokens)
        torch.cuda.synchronize()
        twice.replay()
        torch.cuda.synchronize()
    for t in range(n):
        small.copy_(part[0][:, :, t:t + 1])
        torch.cuda.synchronize()
        few.replay()
        torch.cuda.synchronize()
    mixed.append(part[1])
    ref = want.draft(k, L)
    assert int(ref["length"].sum()) > 0
    b = want.dump_matches(k, cap=1 << 22)
    for ix in (by_graph, mixed):
        _same(ix.draft(k, L), ref)
        a = ix.dump_matches(k, cap=1 << 22)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert ix.status() == 0


@pytest.mark.parametrize("edits", (0, 1))
def test_a_bulk_append_to_a_full_index_ends(edits):
    """A single captured step writes its ends to the other buffer: replayed again and again it files
    the same positions, until the index has no slot left.  A bulk append to such an index ends (what
    it finds no slot for is dropped), and a reset makes the handle whole again."""
    print("bulk, full index", edits, flush=True)
    rng = np.random.default_rng(edits)
    P, N, T, V, k, L = 40, 16, 64, 5, 3, 4
    make = lambda: binding.Index(P, N, T, V, k, L, 0.5, 0, binding.MATCH_INDEX, device="cuda:0", max_edits=edits)
    past, more = _put(_tokens(rng, P, N, 8, V)), _put(_tokens(rng, P, N, 24, V))
    ix = make()
    ix.append(past)
    token = past[:, :, 0].contiguous()
    graph, _ = _captured(lambda: ix.step(token, None, None, 1, k, L))
    for turn in range(300):                                # 16 postings a replay, or up to 64; 1920 or 7680 slots
        token.copy_(past[:, :, turn % 8])
        graph.replay()
    torch.cuda.synchronize()
    ix.append(more)
    torch.cuda.synchronize()
    ix.reset()
    fresh = make()
    for index in (ix, fresh):
        index.append(more)
    _same(ix.draft(k, L), fresh.draft(k, L))
    assert ix.status() == 0


@pytest.mark.parametrize("paths,max_len", [(4, 64), (4, 128), (4, 256), (5, 700)])      # 32 .. 512 buckets
@pytest.mark.parametrize("call", ["append", "step"])
def test_a_gram_that_fills_its_index_takes_every_slot(paths, max_len, call):
    """Replays of a single captured step file a gram again and again, until all slots but a few of its
    index are taken: what is appended then finds those few, and is found there."""
    print("every slot", paths, max_len, call, flush=True)
    buckets = 4
    while buckets * 8 < paths * max_len:
        buckets *= 2
    only = lambda *rows: _put(np.isin(np.arange(paths), rows).astype(np.int32))
    past = _put(np.full((1, paths, 6), 7, dtype=np.int32))
    others = _put(np.tile(np.array([7, 7, 7, 5, 6, 9, 8], dtype=np.int32), (1, paths, 1)))
    token = past[:, :, 0].contiguous()

    def last(ix):                                          # of path 0, from what the others append last
        n = others.shape[2] if call == "append" else 3     # (no row but path 0, which passes over its own, asks for (777))
        ix.append(others[:, :, :n].contiguous(), None, only(*range(1, paths)).reshape(1, paths) * n)
        for t in range(n, others.shape[2]):
            ix.step(others[:, :, t].contiguous(), None, only(*range(1, paths)).reshape(1, paths), 1, 3, 4)
        out = ix.draft(3, 4)
        return {key: out[key][0, 0] for key in KEYS}, ix.status()

    make = lambda: binding.Index(1, paths, max_len, 10, 3, 4, 1.0, 0, binding.MATCH_INDEX, device="cuda:0")
    ix, fresh = make(), make()
    one = only(0).reshape(1, paths)
    for index in (ix, fresh):
        index.append(past, None, one * 6)
    graph, _ = _captured(lambda: ix.step(token, None, one, 1, 3, 4))
    fresh.step(token, None, one, 1, 3, 4)
    # three of path 0's own before; of each other path (777), (775), (756), (569), and a rest
    for _ in range(buckets * 15 - 3 - 4 * (paths - 1) - 4):
        graph.replay()
    torch.cuda.synchronize()
    (got, status), (want, status1) = last(ix), last(fresh)
    _same(got, want)
    assert got["tokens"][:4].tolist() == [5, 6, 9, 8] and status == status1 == 0

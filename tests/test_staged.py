"""Replays of many small problems in one launch, a problem's histories in a workgroup's LDS: the same as a
launch per step."""
import numpy as np
import pytest
import torch

from paper_2503_05330_amd import binding

pytestmark = pytest.mark.gpu
KEYS = ("tokens", "length", "token_scores", "path_scores", "accept")


def _inputs(problems, paths, T, vocab, noise, seed):
    rng = np.random.default_rng(seed)
    pool = rng.integers(0, vocab, size=(problems, 1, 12, 10)).astype(np.int32)      # segments in any order
    order = rng.integers(0, 12, size=(problems, paths, T // 10 + 1))
    if noise < 0.1:
        order[:] = order[:, :1]                                                     # ... in the same one
    tokens = np.take_along_axis(np.repeat(pool, paths, axis=1), order[..., None], axis=2).reshape(problems, paths, -1)[:, :, :T]
    tokens = np.where(rng.random(tokens.shape) < noise, rng.integers(0, vocab, size=tokens.shape), tokens).astype(np.int32)
    probs = (rng.integers(0, 5, size=tokens.shape) / 4.0).astype(np.float32)        # (equal weights)
    return tokens, probs


def _run(problems, paths, T, steps, query, draft, vocab, mode, warm, noise, calls=1, ragged=True, options=True, index=None,
         per_launch=0):
    """`calls` replays one after the other, then a draft; all outputs and the status."""
    dev = torch.device("cuda:0")
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    tokens, probs = _inputs(problems, paths, T, vocab, noise, problems + paths + steps)
    ix = index or binding.Index(problems, paths, T, vocab, query, draft, 0.7, mode, binding.MATCH_INDEX, device=dev)
    if per_launch:
        ix.set_steps_per_launch(per_launch)
    if warm:
        counts = np.where(np.arange(paths) % 5 == 4, warm // 3, warm) if ragged else np.full(paths, warm)
        counts = np.broadcast_to(counts, (problems, paths)).astype(np.int32)
        ix.append(put(tokens[:, :, :warm]), put(probs[:, :, :warm]), put(counts), warm)
    outs = []
    for c in range(calls):
        at = (warm + c * steps + np.arange(steps)) % T
        aim = (at[:, None] + 1 + np.arange(draft)) % T
        targets = put(tokens[:, :, aim].transpose(2, 0, 1, 3)) if options else None
        p = put(probs[:, :, at].transpose(2, 0, 1)) if options else None
        outs.append(ix.replay(steps, put(tokens[:, :, at].transpose(2, 0, 1)), p, query, draft, targets=targets, scores=options))
    outs.append(ix.draft(query, draft))
    return outs, ix.status()


def _same(a, b):
    for x, y in zip(a, b):
        for key in KEYS:
            if x.get(key) is not None or y.get(key) is not None:
                assert torch.equal(x[key], y[key]), key


# cells a path not a multiple of four; the most cells that fit; more paths than a wave has lanes; several
# workgroups a problem with rows left over; grams of two to eight tokens, drafts of one to sixteen; paths that
# agree in all but 2 % (more matches than are listed: placed by a second pass); two symbols (rows of hundreds of
# matches: left to a wave each, in list after list); short paths; paths that are full before the last step
@pytest.mark.parametrize("problems,paths,T,steps,query,draft,vocab,mode,warm,noise", [
    (64, 16, 1024, 48, 3, 8, 300, 0, 900, 0.2),
    (150, 13, 777, 21, 4, 7, 500, 0, 600, 0.3),
    (9, 16, 1022, 255, 3, 8, 100, 1, 700, 0.3),
    (40, 190, 81, 17, 2, 16, 3000, 0, 40, 0.5),
    (300, 16, 250, 24, 3, 8, 1000, 0, 200, 0.02),
    (300, 16, 250, 23, 3, 15, 1000, 1, 200, 0.02),
    (128, 16, 400, 30, 3, 8, 2, 0, 300, 0.5),
    (70, 31, 512, 16, 8, 1, 40, 0, 400, 0.3),
    (520, 7, 100, 16, 6, 16, 30, 1, 60, 0.3),
    (1000, 2, 100, 25, 4, 5, 50, 0, 0, 0.3),
    (600, 4, 64, 16, 3, 4, 60, 0, 60, 0.3),
])
def test_staged_replay(problems, paths, T, steps, query, draft, vocab, mode, warm, noise):
    print("staged", problems, paths, T, steps, query, draft, vocab, mode, warm, noise, flush=True)
    assert problems * paths * steps >= 1 << 15 and paths * ((T + 3) // 4 * 4) <= 1 << 14
    args = (problems, paths, T, steps, query, draft, vocab, mode, warm, noise)
    calls = min(2, max(1, (T - warm) // steps))
    (a, status), (b, status1) = _run(*args, calls=calls), _run(*args, calls=calls, per_launch=1)
    _same(a, b)
    assert status == status1 and (status == 0 or warm + steps > T)
    assert sum(int(x["length"].sum()) for x in a) > 0


def _shares(problems, paths, T, steps, draft):
    """Workgroups of a problem, 0 where the launches for append and drafts are taken (as the library has it)."""
    cells, rows, drafts = paths * ((T + 3) // 4 * 4), paths * steps, problems * paths * steps
    if drafts < 5 << 10 or paths > 256 or cells > 1 << 14 or draft > 16:
        return 0
    shares = max(min(256 // problems, rows // 128), -(-rows // 384))
    per = -(-rows // shares)
    shares = -(-rows // per)
    groups = problems * shares
    staged = 6000 + -(-groups // 256) * (3000 + 100 * paths * ((T + 511) // 512) + cells // 2 + 23 * per) + 16 * groups
    quads = max(0, drafts - (1 << 15))
    launches = 14000 + (drafts - quads) // 2 + quads // 16 + problems * cells // 1500 + drafts * cells // 41000
    return shares if 20 * staged < 19 * launches else 0


# sizes that take the staged form by its rule, and beside its line: few problems of many shares; most paths a problem may
# have; short paths, from empty and full before the last step; all rows left over by few problems
@pytest.mark.parametrize("shares,problems,paths,T,steps,query,draft,vocab,mode,warm,noise", [
    (26, 4, 16, 1000, 215, 3, 8, 300, 0, 700, 0.2),
    (0, 4, 16, 1000, 213, 3, 8, 300, 0, 700, 0.2),
    (4, 9, 8, 512, 72, 4, 7, 100, 1, 400, 0.3),
    (4, 64, 256, 64, 4, 3, 8, 900, 0, 50, 0.3),
    (4, 64, 190, 81, 6, 2, 16, 3000, 0, 40, 0.5),
    (1, 300, 7, 100, 12, 6, 16, 30, 1, 60, 0.3),
    (1, 256, 2, 100, 15, 4, 5, 50, 0, 0, 0.3),
    (1, 300, 4, 64, 14, 3, 4, 60, 0, 60, 0.3),
    (1, 256, 16, 1000, 4, 3, 8, 300, 0, 900, 0.2),
    (0, 256, 16, 1000, 2, 3, 8, 300, 0, 900, 0.2),
    (8, 20, 16, 1000, 64, 3, 8, 2, 0, 900, 0.5),
])
def test_staged_replay_along_its_rule(shares, problems, paths, T, steps, query, draft, vocab, mode, warm, noise):
    print("staged rule", shares, problems, paths, T, steps, query, draft, vocab, mode, warm, noise, flush=True)
    assert _shares(problems, paths, T, steps, draft) == shares and steps <= max(T // 4, 16)
    args = (problems, paths, T, steps, query, draft, vocab, mode, warm, noise)
    (a, status), (b, status1) = _run(*args), _run(*args, per_launch=1)
    _same(a, b)
    assert status == status1 and (status == 0 or warm + steps > T)
    assert sum(int(x["length"].sum()) for x in a) > 0


def _matches(tokens, lens, steps, query):
    """Matches of every row (step by step, path by path) of one problem; tokens: its paths with the steps' tokens."""
    where, rows = {}, []
    for j, path in enumerate(tokens):
        for e in range(query, lens[j] + steps):
            where.setdefault(tuple(path[e - query:e]), []).append((j, e))
    for t in range(steps):
        for i, path in enumerate(tokens):
            end = lens[i] + t + 1
            rows.append(sum(j != i and e < lens[j] + t + 1 for j, e in where.get(tuple(path[end - query:end]), ())))
    return np.array(rows)


def test_matches_without_room_in_a_share_that_ends_within_a_wave():
    """More matches than are placed, and lanes without a row behind them: what is left over are rows of the share."""
    problems, paths, T, steps, query, warm, noise = 300, 24, 200, 15, 3, 110, 0.03
    tokens, _ = _inputs(problems, paths, T, 1000, noise, problems + paths + steps)
    lens, placed = np.where(np.arange(paths) % 5 == 4, warm // 3, warm), []
    for p in (0, problems - 1):
        filed = [np.concatenate([tokens[p, i, :lens[i]], tokens[p, i, warm:warm + steps]]) for i in range(paths)]
        placed.append(_matches(filed, lens, steps, query))
        # one share; more than 6144 matches of rows that could be drafted, few enough that none gives up
        assert len(placed[-1]) == 360 and placed[-1].max() <= 256 and 6144 < placed[-1].sum() <= 1 << 14
    print("without room", [int(x.sum()) for x in placed], flush=True)
    args = (problems, paths, T, steps, query, 8, 1000, 0, warm, noise)
    (a, status), (b, status1) = _run(*args, calls=2), _run(*args, calls=2, per_launch=1)
    _same(a, b)
    assert status == status1 == 0


def test_staged_replay_without_options():
    """No probabilities, targets and scores."""
    args = (200, 16, 300, 24, 3, 8, 200, 0, 200, 0.2)
    _same(_run(*args, options=False)[0], _run(*args, options=False, per_launch=1)[0])


def test_staged_replay_behind_a_reset_and_captured():
    """The same handle over and over: rows left over or none, and from a graph, replay after replay."""
    dev, args = torch.device("cuda:0"), (128, 16, 400, 24, 3, 8, 2, 0, 300, 0.5)
    ix = binding.Index(128, 16, 400, 1000, 3, 8, 0.7, 0, binding.MATCH_INDEX, device=dev)
    want = {v: _run(*args[:6], v, *args[7:], per_launch=1)[0] for v in (2, 1000)}
    for vocab in (2, 1000, 2, 2, 1000):
        ix.reset()
        _same(_run(*args[:6], vocab, *args[7:], index=ix)[0], want[vocab])
    tokens, probs = (torch.from_numpy(x).to(dev) for x in _inputs(128, 16, 400, 2, 0.5, 1))
    past, past_probs = tokens[:, :, :200].contiguous(), probs[:, :, :200].contiguous()
    now, now_probs = (x[:, :, 200:222].permute(2, 0, 1).contiguous() for x in (tokens, probs))
    out = ix.replay(22, now, now_probs, 3, 8)              # (buffers of the graph)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ix.replay(22, now, now_probs, 3, 8, out=out)
    for again in range(3):
        eager = binding.Index(128, 16, 400, 1000, 3, 8, 0.7, 0, binding.MATCH_INDEX, device=dev)
        eager.set_steps_per_launch(1)
        for index in (ix, eager):
            index.reset()
            index.append(past, past_probs)
        for _ in range(1 + again):                         # (goes on from where it was)
            graph.replay()
            torch.cuda.synchronize()
            want_out = eager.replay(22, now, now_probs, 3, 8)
            for key in KEYS[:4]:
                assert torch.equal(out[key], want_out[key]), (again, key)


# all rows left over, in lists of 1024 rows an XCD (a wave a workgroup takes them) and of more (all four): every
# wave of that launch has the lists' counts before they are zeroed for the next replay, so no row stays as it was
@pytest.mark.parametrize("problems,steps", [(20, 25), (20, 60), (64, 30)])
def test_every_row_left_over_is_drafted(problems, steps):
    print("left over", problems, steps, flush=True)
    dev = torch.device("cuda:0")
    tokens, probs = (torch.from_numpy(x).to(dev) for x in _inputs(problems, 16, 1000, 2, 0.5, 3))
    past, past_probs = tokens[:, :, :900].contiguous(), probs[:, :, :900].contiguous()
    now, now_probs = (x[:, :, 900:900 + steps].permute(2, 0, 1).contiguous() for x in (tokens, probs))
    outs = []
    for per_launch in (1, 0):
        ix = binding.Index(problems, 16, 1000, 2, 3, 8, 1.0, 0, binding.MATCH_INDEX, device=dev)
        if per_launch:
            ix.set_steps_per_launch(per_launch)
        for _ in range(1 if per_launch else 6):
            ix.reset()
            ix.append(past, past_probs)
            out = {"tokens": torch.full((steps, problems, 16, 8), -7, dtype=torch.int32, device=dev),
                   "length": torch.full((steps, problems, 16), -7, dtype=torch.int32, device=dev),
                   "token_scores": torch.full((steps, problems, 16, 8), -7.0, device=dev),
                   "path_scores": torch.full((steps, problems, 16), -7.0, device=dev)}
            ix.replay(steps, now, now_probs, 3, 8, out=out)
            outs.append(out)
    for out in outs[1:]:
        _same(outs[:1], [out])

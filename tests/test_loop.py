"""csd_accept_loop with all its steps in one launch (sixteen lanes a path) against a launch per step
(csd_set_steps_per_launch 1), at the sizes and inputs where the two differ; the oracle checks the loop in
test_gpu_parity.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2503_05330_amd import binding


def _inputs(kind, P, N, T, rng):
    if kind == "phrases":                                  # paths share phrases in different order
        phrases = rng.integers(0, 500, (P, 24, 12))
        order = rng.integers(0, 24, (P, N, -(-T // 12)))
        tok = np.concatenate([np.stack([phrases[p][order[p, i]].reshape(-1)[:T] for i in range(N)])[None] for p in range(P)])
        tok = np.where(rng.random((P, N, T)) < 0.05, rng.integers(0, 500, (P, N, T)), tok)
    elif kind.startswith("agree"):                         # paths agree, each gram so many times in each of them
        period = -(-T // int(kind[5:]))
        tok = np.broadcast_to(rng.integers(0, 500, (P, 1, period)), (P, N, period))
        tok = np.tile(tok, (1, 1, int(kind[5:])))[:, :, :T]
        tok = np.where(rng.random((P, N, T)) < 0.03, rng.integers(0, 500, (P, N, T)), tok)
    elif kind == "constant":                               # thousands of matches
        tok = np.full((P, N, T), 7)
    elif kind == "periodic":                               # each gram many times in a path
        tok = np.broadcast_to(np.arange(T) % 40, (P, N, T)).copy()
        tok = np.where(rng.random((P, N, T)) < 0.1, rng.integers(0, 40, (P, N, T)), tok)
    else:                                                  # few symbols: long chains, many candidates
        tok = rng.integers(0, 4, (P, N, T))
    return tok.astype(np.int32), rng.random((P, N, T), dtype=np.float32)


def _run(tok, probs, lens, steps, kmax, L, alpha, mode, per_launch, vocab=600):
    P, N, T = tok.shape
    dev = torch.device("cuda:0")
    d_tok, d_pr = torch.from_numpy(tok).to(dev), None if probs is None else torch.from_numpy(probs).to(dev)
    ix = binding.Index(P, N, T, vocab, kmax, L, alpha, mode, binding.MATCH_INDEX, device=dev)
    if per_launch:
        ix.set_steps_per_launch(per_launch)
    n0 = int(lens.max())
    if n0 > 0:
        ix.append(d_tok[:, :, :n0].contiguous(), None if d_pr is None else d_pr[:, :, :n0].contiguous(),
                  torch.from_numpy(lens.astype(np.int32)).to(dev), n0)
    outs = [ix.accept_loop(steps, d_tok, d_pr, kmax, L), ix.accept_loop(3, d_tok, d_pr, kmax, L)]   # goes on from the first
    status = ix.status()
    # the state that it leaves: a draft, and what more tokens make of the index
    outs.append(ix.draft(kmax, L))
    more = torch.from_numpy(np.ascontiguousarray(tok[:, ::-1, :5])).to(dev)
    ix.append(more, None, torch.ones((P, N), dtype=torch.int32, device=dev) * 5, 5)
    outs.append(ix.draft(kmax, L))
    rows = [{k: v.cpu().numpy() for k, v in o.items() if torch.is_tensor(v) and k != "_scratch"} for o in outs]
    return rows, status


@pytest.mark.parametrize("kind,P,N,T,steps,kmax,L", [
    ("phrases", 1, 16, 400, 60, 3, 8), ("phrases", 3, 13, 300, 41, 4, 16), ("phrases", 2, 1, 200, 9, 3, 5),
    ("phrases", 260, 2, 130, 12, 2, 1), ("phrases", 1, 4, 200, 200, 3, 8), ("phrases", 2, 5, 257, 30, 3, 15),
    ("phrases", 1, 8, 300, 33, 4, 9), ("phrases", 3, 6, 120, 20, 3, 1), ("constant", 1, 16, 60, 8, 3, 8),
    ("periodic", 1, 16, 300, 40, 3, 16), ("periodic", 2, 7, 300, 40, 3, 7), ("symbols", 2, 16, 256, 25, 4, 8),
    ("phrases", 1, 17, 300, 40, 3, 8), ("phrases", 64, 32, 200, 12, 4, 16), ("periodic", 64, 29, 120, 8, 3, 8),
    # queries of two tokens, from 512 rows on
    ("phrases", 130, 4, 100, 12, 2, 8), ("symbols", 128, 4, 60, 10, 2, 16), ("phrases", 64, 8, 100, 12, 2, 16),
    ("phrases", 40, 13, 100, 12, 2, 1), ("phrases", 32, 16, 100, 12, 2, 9), ("phrases", 64, 30, 120, 12, 2, 5),
    # one to four matches a lane, and more: 15, 16 / 17, 32 / 33 .. 36, 60, 64 / 65, 69 matches where all agree
    ("agree1", 2, 16, 300, 30, 3, 8), ("agree1", 3, 18, 200, 20, 3, 16), ("agree2", 1, 9, 300, 30, 3, 8),
    ("agree2", 2, 17, 300, 20, 4, 7), ("agree3", 1, 13, 300, 25, 3, 12), ("agree4", 2, 16, 400, 20, 3, 8),
    ("agree4", 1, 17, 400, 20, 3, 16), ("agree3", 1, 24, 300, 20, 4, 5), ("agree12", 2, 6, 400, 20, 3, 8),
    ("agree40", 1, 4, 400, 20, 3, 3)])
def test_one_launch_equals_a_launch_per_step(kind, P, N, T, steps, kmax, L):
    assert kmax > 2 or P * N >= 512                        # (else both are a launch per step, as with more than 24 paths of few problems)
    assert N <= 24 or P >= 64
    print("loop", kind, P, N, T, steps, kmax, L, flush=True)
    rng = np.random.default_rng(P * 1000 + N * 10 + L)
    tok, probs = _inputs(kind, P, N, T, rng)
    half = rng.integers(0, T // 2 + 1, (P, N))
    half[:, 0] = T - 4                                     # one path is full after a few steps
    for lens, pr, alpha, mode in ((half, probs, 1.0, 0), (half, None, 0.5, 1), (np.zeros((P, N), np.int64), probs, 0.25, 0)):
        want, status = _run(tok, pr, lens, steps, kmax, L, alpha, mode, 1)
        got, status_got = _run(tok, pr, lens, steps, kmax, L, alpha, mode, 0)
        assert status_got == status
        for part, (g, w) in enumerate(zip(got, want)):
            assert g.keys() == w.keys()
            for name in w:
                assert np.array_equal(g[name], w[name]), (kind, part, name)


def test_tokens_out_of_range_and_a_captured_loop():
    rng = np.random.default_rng(5)
    tok, probs = _inputs("phrases", 1, 16, 300, rng)
    tok[0, 3, 104] = 600                                   # (the vocabulary has 600 tokens)
    lens = np.full((1, 16), 100)
    assert _run(tok, probs, lens, 10, 3, 8, 1.0, 0, 0)[1] == _run(tok, probs, lens, 10, 3, 8, 1.0, 0, 1)[1] == binding.STATUS_TOKEN_RANGE
    # a captured loop of an even number of steps goes on at every replay, like the calls one after the other
    dev = torch.device("cuda:0")
    tok, probs = _inputs("phrases", 2, 16, 400, rng)
    d_tok, d_pr = torch.from_numpy(tok).to(dev), torch.from_numpy(probs).to(dev)
    def index():
        ix = binding.Index(2, 16, 400, 600, 3, 8, device=dev)
        ix.append(d_tok[:, :, :100].contiguous(), d_pr[:, :, :100].contiguous())
        return ix
    plain, ix = index(), index()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = ix.accept_loop(6, d_tok, d_pr, 3, 8)
    for _ in range(4):
        want = plain.accept_loop(6, d_tok, d_pr, 3, 8)
        graph.replay()
        torch.cuda.synchronize()
        for name in ("tokens", "length", "accept", "path_len"):
            assert torch.equal(out[name], want[name]), name
        d_tok.clone().sum().item()                         # work of the program's own between the replays


def test_more_paths_than_a_grid_of_fills_has_workgroups():
    """2^24 paths: a workgroup for each would be a grid of 2^32 threads, which is refused."""
    P, N, T = 1 << 20, 16, 8
    print("loop, many paths", P, N, T, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k, L, steps = 3, 1, 3
    phrase = torch.randint(0, 40, (P, 1, T), generator=gen, device="cuda", dtype=torch.int32)
    tok = torch.where(torch.rand((P, N, T), generator=gen, device="cuda") < 0.1, phrase + 1, phrase).contiguous()
    lens = torch.randint(0, T // 2 + 1, (P, N), generator=gen, device="cuda", dtype=torch.int32)
    outs = []
    for per_launch in (1, 0):
        ix = binding.Index(P, N, T, 64, k, L, 1.0, 0, binding.MATCH_INDEX, device="cuda:0")
        if per_launch:
            ix.set_steps_per_launch(per_launch)
        ix.append(tok[:, :, :T // 2].contiguous(), None, lens)
        outs.append((ix.accept_loop(steps, tok, None, k, L), ix.draft(k, L), ix.status()))
        del ix
    (loop, then, status), (loop_got, then_got, status_got) = outs
    assert int(loop["accept"].sum()) > 0 and status == status_got
    for name in ("tokens", "length", "accept", "path_len"):
        assert torch.equal(loop_got[name], loop[name]), name
    for name in ("tokens", "length", "token_scores", "path_scores"):
        assert torch.equal(then_got[name], then[name]), name

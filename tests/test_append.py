"""Appends of many tokens per call against the oracle: the kernel with a thread per new position,
the one with a workgroup per problem (24 problems and more), with the buckets and with the fill
counts only in LDS, on an empty and on a filled index."""
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
    rng = np.random.default_rng(problems * 1000 + vocab + query + edits)
    N, T, L = 5, 720, 6
    tokens = rng.integers(0, vocab, size=(problems, N, T)).astype(np.int32)
    motif = rng.integers(0, vocab, size=(problems, 1, 60)).astype(np.int32)
    shared = rng.random((problems, N, T // 60)) < 0.5          # segments that the paths have in common
    tokens = np.where(np.repeat(shared, 60, axis=2), np.tile(motif, (1, 1, T // 60)), tokens)
    probs = rng.random(tokens.shape).astype(np.float32)
    dev = torch.device("cuda:0")
    ix = binding.Index(problems, N, T, vocab, query, L, 0.5, 0, flags, device=dev, max_edits=edits)
    at = np.zeros((problems, N), dtype=np.int64)
    for turn, n in enumerate(sizes):
        print("append", problems, vocab, query, edits, flags, n, ragged, flush=True)
        counts = rng.integers(0, n + 1, size=at.shape) if ragged else np.full(at.shape, n)
        idx = np.minimum(at[..., None] + np.arange(n), T - 1)
        step = lambda a: torch.from_numpy(np.ascontiguousarray(np.take_along_axis(a, idx, axis=2))).to(dev)
        ix.append(step(tokens), None if turn % 2 else step(probs),
                  torch.from_numpy(counts.astype(np.int32)).to(dev) if ragged else None, n)
        if turn % 2:                                           # no probabilities: all 1
            for p, i in np.ndindex(at.shape):
                probs[p, i, at[p, i]:at[p, i] + counts[p, i]] = 1.0
        at += counts
        lens = at.astype(np.int32)
        out = ix.draft(query, L)
        want = oracle.draft_all(tokens, probs, lens, query, L, 0.5, 0, eps=edits)
        assert np.array_equal(out["tokens"].cpu().numpy(), want["draft"])
        assert np.array_equal(out["length"].cpu().numpy(), want["draft_len"])
        assert np.array_equal(out["path_scores"].cpu().numpy(), want["path_scores"].astype(np.float32))
    je, off = ix.dump_matches(query, cap=1 << 22)
    for r in range(0, problems * N, 1 if problems == 1 else 7):
        p, i = divmod(r, N)
        assert np.array_equal(je[off[r]:off[r + 1]], oracle.matches(tokens[p], lens[p], i, query, eps=edits))
    assert ix.status() == 0


def test_an_append_that_does_not_fit_is_clipped(oracle):
    """Counts beyond max_len: clipped, with the status bit, by both kernels."""
    rng = np.random.default_rng(9)
    for problems in (1, 24):
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

"""What a program that drafts with this framework has it do, as cases to be timed.

A pass is one served request (or one batch of them): the pool is emptied, the tokens that
every path has generated so far are appended in one call, and the decode loop goes on from
there, step by step, with the calls of `binding.Index` that such a program makes:

  steps      one `step` per decode step (append, draft and accept in one launch), its outputs
             newly allocated by each call: a serving loop that runs the model in between
  calls      `append`, `draft` and `accept` for each step: a loop that keeps them apart
  ragged     `step` with up to `offer` tokens a path and a count for each path: what a loop
             appends after its drafts were accepted to different lengths
  replay     `replay`: the steps of recorded traces, one token a path and step
  loop       `accept_loop`: propose, verify, accept, with each path's own future as the model
  prefill    the append of whole histories of different lengths, and one draft of every path
             from them

The inputs have the structure of parallel samples of one prompt: the paths of a problem share
segments of a common pool in different order, with tokens substituted and inserted; token ids
follow a Zipf law; tokens of the pool were sampled with probability 0.5 .. 1 and the others
with 0.01 .. 0.3.  They are drawn on the GPU, from the seed alone.
"""
import math

import torch

from paper_2503_05330_amd import binding

_KEYS = ("call", "problems", "paths", "max_len", "steps", "vocab", "query", "draft", "max_edits",
         "score_mode", "alpha", "pool", "probs", "segments", "seg_lo", "seg_hi", "zipf", "sub", "ins", "offer")
_POOLS = {"dag": binding.POOL_DAG, "tree": binding.POOL_TREE, "list": binding.POOL_LIST}


def _case(name, call, problems, paths, max_len, steps, vocab=32000, query=3, draft=8, max_edits=0, score_mode=0,
          alpha=1.0, pool="dag", probs=True, segments=256, seg_lo=8, seg_hi=32, zipf=1.1, sub=0.05, ins=0.0,
          offer=1):
    values = (call, problems, paths, max_len, steps, vocab, query, draft, max_edits, score_mode, alpha, pool, probs,
              segments, seg_lo, seg_hi, zipf, sub, ins, offer)
    c = dict(zip(_KEYS, values))
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest request: four short samples, a serving loop that calls once per token.
        # Latency, launches and the host's part are all there is to it.
        _case("steps_4x256", "steps", 1, 4, 256, 12, draft=5, segments=64, seg_hi=24),
        # sixteen samples of 1024 tokens, the size that the latency of a step is quoted on:
        # recorded traces at (nearly) full history
        _case("replay_16x1024", "replay", 1, 16, 1024, 64),
        # the same samples where the loop appends what was accepted: 1 .. 9 tokens a path and step
        _case("ragged_16x1024", "ragged", 1, 16, 1024, 12, offer=9),
        # more and longer samples, a large vocabulary, queries of four tokens, tokens inserted
        _case("replay_32x2048", "replay", 1, 32, 2048, 64, vocab=128256, query=4, draft=10, segments=512, seg_hi=48,
              zipf=1.05, sub=0.08, ins=0.10),
        # the longest histories of one problem and the longest usual draft; samples that agree little
        _case("replay_64x4096", "replay", 1, 64, 4096, 48, vocab=152064, query=4, draft=16, segments=2048, seg_lo=4,
              seg_hi=64, zipf=1.0, sub=0.20),
        # a server's batch: 64 problems in one launch
        _case("replay_64_problems", "replay", 64, 16, 1024, 48),
        # the largest batch: 1024 problems, 16384 rows in a launch
        _case("replay_1024_problems", "replay", 1024, 16, 1024, 24),
        # matching that tolerates one edit, which the method's own experiments use: short queries
        _case("one_edit_16x1024", "replay", 1, 16, 1024, 32, max_edits=1),
        # and queries of four tokens in long histories
        _case("one_edit_64x4096", "replay", 1, 64, 4096, 24, vocab=152064, query=4, draft=16, max_edits=1,
              segments=2048, seg_lo=4, seg_hi=64, zipf=1.0, sub=0.20),
        # the accept-driven decode loop
        _case("loop_16x1024", "loop", 1, 16, 1024, 48),
        # histories handed over as a whole: a request that is resumed, or moved from another server
        _case("prefill_64x4096", "prefill", 1, 64, 4096, 1, vocab=152064, query=4, draft=16, segments=2048, seg_lo=4,
              seg_hi=64, zipf=1.0, sub=0.20),
        # odd sizes and the options: three calls per step, a tree of candidates, half of the
        # weight from frequencies, no probabilities recorded
        _case("calls_3x13x777_tree", "calls", 3, 13, 777, 12, vocab=50021, draft=7, alpha=0.5, pool="tree",
              probs=False, segments=150, sub=0.07, ins=0.03),
    ]


def _spread(rng, lo, hi):
    """A whole number in lo .. hi, evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(("steps", "calls", "ragged", "replay", "replay", "replay", "loop", "prefill"))
    one_edit = call != "prefill" and rng.random() < 0.25
    paths = _spread(rng, 2, 64)
    max_len = _spread(rng, 128, 4096)
    # what a launch has to hold: 2^23 positions, one-edit matching 2^18 (its scans read them all)
    most = (1 << 18 if one_edit else 1 << 23) // (paths * max_len)
    problems = _spread(rng, 1, max(1, min(1024, most))) if rng.random() < 0.5 else 1
    query = rng.choice((3, 3, 4, 5)) if one_edit else rng.choice((2, 3, 3, 4, 4, 6))
    steps = {"steps": 12, "calls": 12, "ragged": 12, "prefill": 1}.get(call) or rng.randint(12, 24)
    draft = rng.randint(1, 16)
    seg_lo = rng.randint(4, 12)
    return _case("", call, problems, paths, max_len, steps,
                 vocab=_spread(rng, 8000, 152064), query=query, draft=draft, max_edits=int(one_edit),
                 score_mode=int(rng.random() < 0.2), alpha=rng.choice((1.0, 1.0, 0.5, 0.25)),
                 pool=rng.choice(("dag", "dag", "dag", "dag", "tree", "list")), probs=rng.random() < 0.75,
                 segments=max(16, paths * max_len // rng.randint(40, 130)), seg_lo=seg_lo,
                 seg_hi=seg_lo + rng.randint(8, 52), zipf=rng.choice((1.0, 1.05, 1.1)),
                 sub=rng.uniform(0.03, 0.2), ins=rng.choice((0.0, 0.0, 0.1)),
                 offer=min(draft + 1, max_len // (2 * steps)) if call == "ragged" else 1)


def _paths(case, gen):
    """Tokens int32 and probabilities float32 of all paths, [P][N][max_len]."""
    P, N, T, V = case["problems"], case["paths"], case["max_len"], case["vocab"]
    S, lo, hi = case["segments"], case["seg_lo"], case["seg_hi"]
    kw = dict(generator=gen, device="cuda")
    law = torch.arange(1, V + 1, dtype=torch.float64, device="cuda") ** -case["zipf"]
    law = (law.cumsum(0) / law.sum()).float()
    pool = torch.searchsorted(law, torch.rand((P, S * hi), **kw)).clamp_(max=V - 1).int()
    seg_len = torch.randint(lo, hi + 1, (P, S), **kw)
    used = -(-T // lo)                                   # segments that surely fill a path
    order = torch.rand((P, N, S), **kw).argsort(-1)      # every path's own order of the pool
    if used > S:                                         # a small pool: drawn again and again
        order = torch.randint(0, S, (P, N, used), **kw)
    order = order[:, :, :used].contiguous()
    ends = seg_len[:, None, :].expand(P, N, S).gather(2, order).cumsum(-1)
    noise = torch.rand((P, N, T), **kw) < case["sub"]
    extra = torch.rand((P, N, T), **kw) < case["ins"]    # inserted tokens push the rest back
    noise |= extra
    at = ((~extra).cumsum(-1) - 1).clamp_(min=0)         # place in the path without them
    nth = torch.searchsorted(ends, at, right=True).clamp_(max=order.shape[2] - 1)
    begin = torch.where(nth > 0, ends.gather(2, (nth - 1).clamp_(min=0)), 0)
    cell = order.gather(2, nth) * hi + (at - begin)
    tokens = pool[:, None, :].expand(P, N, S * hi).gather(2, cell)
    tokens = torch.where(noise, torch.randint(0, V, (P, N, T), dtype=torch.int32, **kw), tokens)
    u = torch.rand((P, N, T), **kw)
    probs = torch.where(noise, 0.01 + 0.29 * u, 0.5 + 0.5 * u)
    return tokens, probs


def _warm(case):
    """Tokens a path has before the timed part's first step."""
    if case["call"] == "prefill":
        return case["max_len"]
    return max(0, case["max_len"] - case["steps"] * case["offer"])


def prepare(case, seed):
    P, N, T, L, S = case["problems"], case["paths"], case["max_len"], case["draft"], case["steps"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    tokens, probs = _paths(case, gen)
    warm, call, n = _warm(case), case["call"], case["offer"]
    if call == "loop":
        warm = T // 2                                    # the loop advances by what it accepts
    s = {"case": case, "warm": warm}
    s["index"] = binding.Index(P, N, T, case["vocab"], case["query"], L, case["alpha"], case["score_mode"],
                               max_edits=case["max_edits"], pool_mode=_POOLS[case["pool"]])
    keep = (lambda t: t.contiguous()) if case["probs"] else (lambda t: None)
    s["past"] = tokens[:, :, :warm].contiguous()
    s["past_probs"] = keep(probs[:, :, :warm])
    if call == "loop":
        s["future"], s["future_probs"] = tokens, keep(probs)
        return s
    if call == "prefill":
        s["counts"] = torch.randint(T // 2, T + 1, (P, N), generator=gen, device="cuda", dtype=torch.int32)
        return s
    # what the steps append, and each path's own next tokens as the targets of its drafts
    later = torch.cat([tokens[:, :, warm:], torch.full((P, N, L), -1, dtype=torch.int32, device="cuda")], 2)
    later_probs = probs[:, :, warm:]
    if call == "ragged":
        counts = torch.randint(1, n + 1, (S, P, N), generator=gen, device="cuda", dtype=torch.int32)
        starts = counts.cumsum(0) - counts
        x = torch.arange(n, device="cuda")
        room = later_probs.shape[2] - 1
        at = (starts[..., None] + x).clamp_(max=room).permute(1, 2, 0, 3).reshape(P, N, S * n)
        aim = (starts + counts)[..., None] + torch.arange(L, device="cuda")
        aim = aim.clamp_(max=later.shape[2] - 1).permute(1, 2, 0, 3).reshape(P, N, S * L)
        by_step = lambda t, w: t.reshape(P, N, S, w).permute(2, 0, 1, 3).contiguous()
        s["tokens"] = by_step(later.gather(2, at), n)
        s["probs"] = by_step(later_probs.gather(2, at), n) if case["probs"] else None
        s["targets"] = by_step(later.gather(2, aim), L)
        s["counts"] = counts
    else:
        s["tokens"] = later[:, :, :S].permute(2, 0, 1).contiguous()
        s["probs"] = keep(later_probs[:, :, :S].permute(2, 0, 1))
        s["targets"] = later.unfold(2, L, 1)[:, :, 1:S + 1].permute(2, 0, 1, 3).contiguous()
    return s


def run(state):
    case, ix = state["case"], state["index"]
    call, k, L, S = case["call"], case["query"], case["draft"], case["steps"]
    ix.reset()
    ix.append(state["past"], state["past_probs"], state["counts"] if call == "prefill" else None)
    if call == "prefill":
        return ix.draft(k, L)
    if call == "loop":
        out = ix.accept_loop(S, state["future"], state["future_probs"], k, L)
        return {name: out[name] for name in ("tokens", "length", "accept", "path_len")}
    tokens, probs, targets = state["tokens"], state["probs"], state["targets"]
    if call == "replay":
        return ix.replay(S, tokens, probs, k, L, targets=targets)
    outs = []
    for t in range(S):
        p = probs[t] if probs is not None else None
        if call == "calls":
            ix.append(tokens[t], p)
            out = ix.draft(k, L)
            out["accept"] = ix.accept(out["tokens"], out["length"], targets[t], L)
        elif call == "ragged":
            out = ix.step(tokens[t], p, state["counts"][t], case["offer"], k, L, targets=targets[t])
        else:
            out = ix.step(tokens[t], p, None, 1, k, L, targets=targets[t])
        outs.append(out)
    return outs


def work(case):
    """Per appended token: itself and its probability read and stored, its posting.  Per draft:
    the newest tokens of its path, one posting of the index with its continuation, the
    targets read and the outputs written.  No floating-point work: integers are compared,
    looked up and summed."""
    rows = case["problems"] * case["paths"]
    k, L, S = case["query"], case["draft"], case["steps"]
    prob = 4 if case["probs"] else 0
    warm = {"loop": case["max_len"] // 2, "prefill": 0.75 * case["max_len"]}.get(case["call"], _warm(case))
    per_step = {"ragged": (case["offer"] + 1) / 2, "prefill": 0, "loop": 2}.get(case["call"], 1)
    appended = rows * (warm + S * per_step)
    draft = 4 * k + 4 + 8 * L + (8 * L + 8) + (0 if case["call"] == "prefill" else 4 * L + 4)
    moved = appended * (4 + prob + 8 + 4) + rows * S * draft
    return {"bytes": moved, "flops": 0}


def tolerance(case):
    # all sums are exact integers, rounded once to a float: any correct order gives the same bits
    return "exact"

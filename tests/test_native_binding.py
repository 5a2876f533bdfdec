"""The native part of the binding: it takes the usual arguments only, and what it returns is what
the Python part returns and raises."""
import warnings

import numpy as np
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2503_05330_amd import binding


def test_unusual_arguments_are_left_to_python():
    binding.load()
    native, pool = binding._native, (0, 0, -1, 2, 3)
    x = torch.zeros((2, 3, 4), dtype=torch.int32)                          # not on a device
    assert native.append(*pool, 4, x, None, None) is None
    assert native.append(*pool, 4, None, None, None) is None               # tokens are not optional
    assert native.append(*pool, 4.0, x, None, None) is None
    assert native.append(*pool, 1 << 40, x, None, None) is None
    assert native.append(*pool) is None
    assert native.append(*pool, True, x, None, None) is None
    assert native.draft(*pool, 3, -1, True) is None
    assert native.draft(*pool, 3, 4, 1) is None
    assert native.draft(*pool, np.int64(3), 4, True) is None
    assert native.accept(*pool, 4, x, x, x) is None
    assert native.step(*pool, 1, 3, 4, True, x, None, None, None, None) is None
    assert native.replay(*pool, 1, 3, 4, True, x, None, True, None, None) is None
    assert native.reset("", 0, -1, 2, 3) is None
    assert native.reset(0, 0, 500, 2, 3) is None
    assert native.reset(*pool) == binding.ERR_INVALID_ARG                  # no handle


@pytest.mark.gpu
@pytest.mark.parametrize("scores", (True, False))
def test_the_same_from_both_parts(scores):
    dev, P, N, T, k, L, S = torch.device("cuda:0"), 2, 5, 60, 3, 6, 4
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    draw = lambda *shape: torch.randint(0, 6, shape, generator=gen, device=dev, dtype=torch.int32)
    past, tokens, targets = draw(P, N, 40), draw(S, P, N), draw(S, P, N, L)
    probs = torch.rand((S, P, N), generator=gen, device=dev)

    def outputs(lead=()):
        mk = lambda shape, dt: torch.empty(tuple(lead) + shape, dtype=dt, device=dev)
        return dict(tokens=mk((P, N, L), torch.int32), length=mk((P, N), torch.int32),
                    token_scores=mk((P, N, L), torch.float32) if scores else None,
                    path_scores=mk((P, N), torch.float32) if scores else None)

    results = []
    for native in (True, False):
        ix = binding.Index(P, N, T, 6, k, L, device="cuda" if native else dev)
        give = (lambda *lead: None) if native else lambda *lead: outputs(lead)
        ix.append(past)
        got = [ix.draft(k, L, out=give(), scores=scores)]
        acc = None if native else torch.empty((P, N), dtype=torch.int32, device=dev)
        got.append({"accept": ix.accept(got[0]["tokens"], got[0]["length"], targets[0], L, out=acc)})
        got.append(ix.step(tokens[0], probs[0], None, 1, k, L, out=give(), targets=targets[0], scores=scores))
        got.append(ix.step(tokens[1], None, torch.ones((P, N), dtype=torch.int32, device=dev), 1, k, L, out=give(),
                           scores=scores))
        got.append(ix.replay(S, tokens, probs, k, L, out=give(S), targets=targets, scores=scores))
        kept = torch.empty((S, P, N), dtype=torch.int32, device=dev)
        got.append(ix.replay(S, tokens, None, k, L, out=give(S), targets=targets, accept_out=kept, fused=False, scores=scores))
        assert got[-1]["accept"] is kept
        results.append(got)
        for call, error in ((lambda: ix.append(past.float()), TypeError), (lambda: ix.append(past[:, :, ::2]), TypeError),
                            (lambda: ix.append(past[0], n=40), ValueError), (lambda: ix.append(past.cpu()), TypeError),
                            (lambda: ix.step(None, None, None, 1, k, L, out=give()), binding.CsdError),
                            (lambda: ix.draft(k, L + 1), binding.CsdError), (lambda: ix.draft(k, -1), RuntimeError),
                            (lambda: ix.append(past), binding.CsdError)):
            with pytest.raises(error):
                call()
        ix.reset()
        assert int(ix.draft(k, L, out=give())["length"].sum()) == 0
    for a, b in zip(*results):
        assert list(a) == list(b)
        for key in a:
            if a[key] is None or b[key] is None:
                assert a[key] is None and b[key] is None
                continue
            assert a[key].dtype == b[key].dtype and a[key].shape == b[key].shape and a[key].is_contiguous(), key
            assert torch.equal(a[key], b[key]), key


@pytest.mark.gpu
@pytest.mark.parametrize("P,N,L,S", ((1, 1, 1, 1), (1, 3, 7, 2), (2, 64, 8, 3), (1, 127, 32, 1), (1, 128, 32, 1), (1, 600, 16, 2)))
def test_outputs_of_a_call_lie_apart(P, N, L, S):
    """No output overlaps another, each starts where an allocation would, and one that is kept outlives
    the others."""
    ix = binding.Index(P, N, 64, 50, 3, 32)
    tokens = torch.randint(0, 4, (S, P, N), device="cuda", dtype=torch.int32)
    targets = torch.zeros((S, P, N, L), device="cuda", dtype=torch.int32)
    kept = []
    for mode in (torch.inference_mode(False), torch.inference_mode(True)):
        with mode:
            ix.reset()
            out = ix.replay(S, tokens, None, 3, L, targets=targets)
            assert all(t.is_inference() == torch.is_inference_mode_enabled() for t in out.values())
        spans = sorted((t.data_ptr(), t.data_ptr() + 4 * t.numel()) for t in out.values())
        assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:])) and all(a % 512 == 0 for a, _ in spans)
        for t in out.values():
            assert t.is_contiguous() and t._base is None and not t.requires_grad
            assert t.storage_offset() * 4 + t.numel() * 4 <= t.untyped_storage().nbytes()
        kept.append((out["length"], out["length"].clone()))
        del out, t
        ix.reset()
        ix.replay(S, tokens.flip(0), None, 3, L)         # would take a freed block of the same size
        assert torch.equal(*kept[-1])
    assert torch.equal(kept[0][0], kept[1][0])


@pytest.mark.gpu
@pytest.mark.parametrize("call", ("draft", "step", "replay"))
def test_each_output_has_a_storage_of_its_own(call):
    """What a caller does in place to one output (a resize, a write as out= of another shape, a storage given
    back) leaves the others alone, and a saved output is no larger than itself."""
    P, N, L, S = 2, 3, 5, 2
    ix = binding.Index(P, N, 64, 50, 3, 8)
    tokens = torch.randint(0, 4, (S, P, N), device="cuda", dtype=torch.int32)
    targets = torch.zeros((S, P, N, L), device="cuda", dtype=torch.int32)
    calls = {"draft": lambda: ix.draft(3, L), "step": lambda: ix.step(tokens[0], None, None, 1, 3, L, targets=targets[0]),
             "replay": lambda: ix.replay(S, tokens, None, 3, L, targets=targets)}
    names = list(calls[call]())
    for changed in names:
        for change in (lambda t: t.resize_(4 * t.numel() + 1000).fill_(77),
                       lambda t: torch.full((t.numel() + 500,), 77, out=t, dtype=t.dtype, device="cuda"),
                       lambda t: t.untyped_storage().resize_(0)):
            ix.reset()
            out = calls[call]()
            assert len({t.untyped_storage().data_ptr() for t in out.values()}) == len(names)
            for t in out.values():
                assert t.storage_offset() == 0 and t.untyped_storage().nbytes() == 4 * t.numel()
            before = {name: t.clone() for name, t in out.items()}
            with warnings.catch_warnings():
                warnings.simplefilter("ignore")          # (out= of another shape)
                change(out[changed])
            for name in names:
                assert name == changed or torch.equal(out[name], before[name]), (changed, name)


@pytest.mark.gpu
def test_a_dispatch_mode_sees_every_output():
    class Seen(TorchDispatchMode):
        count = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.count += func is torch.ops.aten.empty.memory_format
            return func(*args, **(kwargs or {}))

    ix = binding.Index(1, 2, 64, 50, 3, 8)
    tokens, targets = torch.zeros((1, 2), device="cuda", dtype=torch.int32), torch.zeros((1, 2, 4), device="cuda", dtype=torch.int32)
    with Seen() as seen:
        ix.step(tokens, None, None, 1, 3, 4, targets=targets)
    assert seen.count == 5

"""A wrapper's scratch comes from the pool of the stream its kernels run on.

torch's caching allocator hands a freed block out again at once on the stream
it belongs to, in that stream's order only. Scratch of a call on another stream
than the current one therefore has to be allocated on that stream: from the
current stream's pool it could be memory that kernels queued there still use.
"""
import contextlib

import pytest
import torch

from paper_2609_40335_amd import dpghost as D

SIDE = 77
B, T, d, V = 2, 3, 8, 16


class _Stream:
    cuda_stream = SIDE


class _Lib:
    """Every entry point succeeds; every size query asks for scratch."""

    def __getattr__(self, name):
        return lambda *a: 512 if name.endswith(("_workspace", "_bytes")) else 0


@pytest.fixture
def allocated(monkeypatch):
    """The current stream (None: the default) at each allocation of scratch."""
    current, seen, empty = [None], [], torch.empty

    @contextlib.contextmanager
    def on(s):
        current.append(s)
        yield
        current.pop()

    def record(*a, **k):
        if k.get("dtype") == torch.uint8:
            seen.append(current[-1])
        return empty(*a, **k)

    lib = _Lib()
    monkeypatch.setattr(D, "lib", lambda: lib)
    monkeypatch.setattr(D, "_dev", lambda t, n: None)
    monkeypatch.setattr(torch, "empty", record)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda p, **k: p)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: type("S", (), {"cuda_stream": 0}))
    return seen


def _calls():
    A, G = torch.zeros(B, T, d), torch.zeros(B, T, d)
    ids, n2, c = torch.zeros(B, T, dtype=torch.int32), torch.zeros(B), torch.ones(B)
    Gz, out, E = torch.zeros(B, T, V), torch.zeros(d, d), torch.zeros(V, d)
    return {
        "norm": lambda s: D.dp_ghost_norm_linear(A, G, n2, stream=s),
        "norms": lambda s: D.dp_ghost_norm_linear_grouped([(A, G)], n2, stream=s),
        "norms_bias": lambda s: D.dp_ghost_norm_linear_bias_grouped([(A, G)], [n2.new_zeros(B, d)], n2,
                                                                    stream=s),
        "norm_embedding": lambda s: D.dp_ghost_norm_embedding(ids, G, V, n2, stream=s),
        "cross": lambda s: D.dp_tied_cross_term(ids, G, A, Gz, V, n2, stream=s),
        "sum": lambda s: D.dp_clipped_grad_sum(A, G, c, out, stream=s),
        "sum_embedding": lambda s: D.dp_clipped_grad_sum(None, G, c, E, ids=ids, V=V, stream=s),
        "vectors": lambda s: D.dp_vector_grads_grouped([(A, G)], [n2.new_zeros(B, d)], n2, stream=s),
        "positions": lambda s: D.dp_ghost_norm_positional(G, n2, stream=s),
    }


@pytest.mark.parametrize("name", sorted(_calls()))
def test_scratch_of_a_call_belongs_to_its_stream(allocated, name):
    _calls()[name](_Stream())
    assert allocated and set(allocated) == {SIDE}
    del allocated[:]
    _calls()[name](None)
    assert allocated and set(allocated) == {None}


def test_group_sums_share_no_scratch_between_streams(allocated):
    """Every sum of a group gets scratch of its own stream's pool, the first call
    and later ones alike, and the group holds one block at most."""
    A, G, c = torch.zeros(B, T, d), torch.zeros(B, T, d), torch.ones(B)
    grp = D.LinearGroup([(A, G)], [torch.zeros(d, d)])
    del allocated[:]
    for s in (_Stream(), None, _Stream()):
        grp.clipped_sum(c, stream=s)
        grp.clipped_sum_noised(c, [0], 1.0, 1.0, B, 1, 1, stream=s)
    assert allocated == [SIDE, SIDE, None, None, SIDE, SIDE]
    held = [v for k, v in vars(grp).items() if k != "ws" and isinstance(v, torch.Tensor)]
    assert len(held) == 1

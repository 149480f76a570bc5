"""RingWalk's native marshalling, as far as it shows without a device: where it is not to be had, and that the module's two
functions take what RingWalk hands them."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd.harness import RingWalk


def host_walk():
    """A walk over tensors in host memory, which either marshalling refuses before anything is enqueued."""
    t = [torch.zeros(1, 2, 8, 64, dtype=torch.bfloat16) for _ in range(4)]
    return RingWalk(t[0], 0.125), [t[1]], [t[2]], t[3]


@pytest.mark.parametrize("error", [FileNotFoundError, ImportError, OSError])
def test_a_walk_without_the_torch_module_is_marshalled_by_itself(error, monkeypatch):
    asked = []

    def missing():
        asked.append(1)
        raise error("not built")

    monkeypatch.setattr(B, "load_torch_module", missing)
    monkeypatch.setattr(B, "_walk_module", None)
    walk, K, V, dO = host_walk()
    for _ in range(2):
        with pytest.raises(ValueError, match="device tensor expected"):
            walk.forward(K, V, [0])
        with pytest.raises(ValueError, match="device tensor expected"):
            walk.backward(K, V, [0], dO)
    assert len(asked) == 1


def test_the_module_takes_what_the_walk_hands_it():
    """Other arguments than declared would be a TypeError, which RingWalk takes for tensors or numbers that are none."""
    module = B.load_torch_module()
    walk, K, V, dO = host_walk()
    common = walk.Q, K, V, [0], walk.scale, walk.causal, walk.q_off, walk.window, walk.kv_heads
    for ws in (None, torch.zeros(16, dtype=torch.uint8)):
        assert module.walk_forward(*common, walk.O_acc, walk.m, walk.l, walk.O, walk.lse, ws, 0) == 1
        assert module.walk_backward(*common, walk.O, dO, walk.lse, walk.D, ws, 0)[0] == 1


def test_an_object_s_own_params_are_asked(monkeypatch):
    walk, K, V, dO = host_walk()
    asked = []

    def params(*args, **kw):
        asked.append(args)
        return RingWalk.params(walk, *args, **kw)

    monkeypatch.setattr(B, "load_torch_module", lambda: pytest.fail("marshalled natively"))
    monkeypatch.setattr(B, "_walk_module", None)
    walk.params = params
    with pytest.raises(ValueError, match="device tensor expected"):
        walk.forward(K, V, [0])
    with pytest.raises(ValueError, match="device tensor expected"):
        walk.backward(K, V, [0], dO)
    assert asked


def test_chunks_that_are_not_dense_are_not_offered(monkeypatch):
    """Every call over sequence-major chunks would convert its tensors only to be refused."""
    walk, K, V, dO = host_walk()
    seq = [torch.zeros(1, 8, 2, 64, dtype=torch.bfloat16).transpose(1, 2)]
    monkeypatch.setattr(B, "load_torch_module", lambda: pytest.fail("offered"))
    monkeypatch.setattr(B, "_walk_module", None)
    with pytest.raises(ValueError, match="device tensor expected"):
        walk.forward(seq, seq, [0])
    with pytest.raises(ValueError, match="device tensor expected"):
        walk.backward(seq, seq, [0], dO)
    monkeypatch.undo()
    with pytest.raises(AttributeError):
        walk.forward([None], [None], [0])

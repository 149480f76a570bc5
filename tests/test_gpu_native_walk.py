"""RingWalk's native marshalling against its own (which lists that are tuples take): the same launches, so the same bits; and what is not
as usual goes to the latter, errors included."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ("f32", dict(H=1, d=64, Nq=256, chunk_rows=[256] * 4)),                                        # no workspace
    ("f32", dict(H=2, d=128, Nq=100, chunk_rows=[300, 500], causal=True, q_off=700)),              # split: a workspace
    ("bf16", dict(H=4, kv_heads=2, d=128, Nq=70, chunk_rows=[90, 1400], causal=True, q_off=1420)),
    ("bf16", dict(H=3, d=96, Nq=129, chunk_rows=[64, 1, 200], window=50, q_off=100)),
    ("bf16", dict(H=2, d=64, Nq=1, chunk_rows=[1])),
]


def taken(walk, monkeypatch):
    """Counts the calls that native code took."""
    count = []
    native = RingWalk._native
    monkeypatch.setattr(RingWalk, "_native", lambda self, *a: (lambda r: (count.append(r is not None), r)[1])(native(self, *a)))
    return count


@pytest.mark.parametrize("dtype,spec", CASES, ids=lambda v: v if isinstance(v, str) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_the_same_bits_as_its_own_marshalling(dtype, spec, monkeypatch):
    case = workloads.make_case(B=1, dtype=dtype, seed=401, device=DEV, **spec)
    results = []
    for of in (list, tuple):
        walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], kv_heads=case.get("kv_heads", 0))
        K, V = of(case["K"]), of(case["V"])
        count = taken(walk, monkeypatch)
        for _ in range(2):                           # (the first pass brings the workspace)
            O, lse = walk.forward(K, V, list(case["k_offs"]))
            dQ, dKs, dVs = walk.backward(K, V, list(case["k_offs"]), case["dO"])
        torch.cuda.synchronize()
        assert count[-2:] == [of is list] * 2
        monkeypatch.undo()
        results.append([O, lse, walk.O_acc, walk.m, walk.l, walk.D, dQ, *dKs, *dVs])
    for a, b in zip(*results):
        assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b)


def test_what_is_not_as_usual_is_marshalled_as_before(monkeypatch):
    case = workloads.make_case(B=1, H=2, d=64, Nq=70, chunk_rows=[80, 60], dtype="bf16", seed=403, device=DEV)
    walk = RingWalk(case["Q"], case["scale"])
    K, V, offs, dO = case["K"], case["V"], list(case["k_offs"]), case["dO"]
    want = [t.clone() for t in walk.forward(K, V, offs)]
    grads = walk.backward(K, V, offs, dO)
    count = taken(walk, monkeypatch)
    seq = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in K], [t.transpose(1, 2).contiguous().transpose(1, 2) for t in V]
    assert all(torch.equal(a, b) for a, b in zip(walk.forward(*seq, offs), want))
    other = dO.transpose(1, 2).contiguous().transpose(1, 2)          # (copied to lie like Q)
    again = walk.backward(K, V, offs, other)
    assert torch.equal(grads[0], again[0]) and all(torch.equal(a, b) for a, b in zip(grads[1] + grads[2], again[1] + again[2]))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert all(torch.equal(a, b) for a, b in zip(walk.forward(K, V, offs), want))
    side.synchronize()
    with pytest.raises(IndexError):
        walk.forward(K, V[:1], offs)
    with pytest.raises(ValueError):
        walk.forward([k.float() for k in K], V, offs)
    with pytest.raises(ValueError):
        walk.forward([k.cpu() for k in K], V, offs)
    with pytest.raises(TypeError):
        walk.forward(K, V, [0.5, 80])
    with pytest.raises(B.BurstError):
        RingWalk(case["Q"], 0.0).forward(K, V, offs)
    assert count == [False, False, True, False, False, False, False, True]


def test_a_row_expanded_to_a_slice_is_refused():
    """Strides of 0 throughout mean a dense tensor in the parameter block: such a Q, which holds one row, is no slice to read."""
    q = torch.randn(64, device=DEV).bfloat16().expand(2, 3, 100, 64)
    K, V = ([torch.randn(2, 3, 70, 64, device=DEV).bfloat16()] for _ in range(2))
    walk = RingWalk(q, 0.125)
    with pytest.raises(ValueError):
        walk.forward(K, V, [0])
    with pytest.raises(ValueError):
        walk.backward(K, V, [0], q)

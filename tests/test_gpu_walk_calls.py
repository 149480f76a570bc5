"""The whole-walk entry points (one call for all chunks) against the same walk chunk by chunk: O, lse, the
state and every gradient bit for bit where the sums come in the same order (fp32 kernels and split keys: to the
rounding of another order), for each kernel family, with empty and invisible chunks in between, chunks of
different pitch in one walk, and more chunks than one launch takes; and against the oracle."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ("bf16", dict(B=1, H=3, d=64, Nq=130, chunk_rows=[64, 1, 200, 33])),
    ("bf16", dict(B=1, H=2, d=128, Nq=257, chunk_rows=[100, 64, 190], causal=True, q_off=90)),
    ("bf16", dict(B=2, H=2, d=80, Nq=65, chunk_rows=[30] * 5, causal=True, q_off=60, window=50)),
    ("bf16", dict(B=1, H=2, d=128, Nq=300, chunk_rows=[200, 128, 70], block=64, pattern="random", density=0.3)),
    ("bf16", dict(B=1, H=4, kv_heads=2, d=64, Nq=100, chunk_rows=[90, 70], block=64, pattern="random", density=0.5,
                  layout="seq")),
    ("bf16", dict(B=1, H=4, kv_heads=2, d=128, Nq=100, chunk_rows=[90, 70], causal=True, q_off=60, layout="packed")),
    ("bf16", dict(B=1, H=2, d=64, Nq=70, chunk_rows=[20] * 37, causal=True, q_off=700)),
    ("f32", dict(B=1, H=2, d=64, Nq=70, chunk_rows=[40, 33, 64])),
    ("bf16", dict(B=1, H=2, d=20, Nq=70, chunk_rows=[40, 33])),
    ("bf16", dict(B=1, H=2, d=128, Nq=300, chunk_rows=[256, 70], block=256, pattern="random", density=0.5)),
    ("bf16", dict(B=1, H=2, d=64, Nq=33, chunk_rows=[1000, 1100])),
]


def chunk_by_chunk(case, walk):
    walk.init()
    masks = case.get("masks") or [None] * len(case["K"])
    for K, V, off, m in zip(case["K"], case["V"], case["k_offs"], masks):
        walk.step(K, V, off, m)
    O, lse = walk.finalize()
    walk.prepare(case["dO"])
    dQ = torch.zeros(walk.Q.shape, device=DEV)
    dKs, dVs = [torch.empty(k.shape, device=DEV) for k in case["K"]], [torch.empty(k.shape, device=DEV) for k in case["K"]]
    for j, (K, V) in enumerate(zip(case["K"], case["V"])):
        B.burst_local_bwd(walk.Q, K, V, walk.O, case["dO"], lse, walk.D, dQ, dKs[j], dVs[j],
                          walk.params(K.shape[2], case["k_offs"][j], masks[j], K), accumulate_dq=True, accumulate_dkv=False)
    return [t.clone() for t in (O, lse, walk.O_acc, walk.m, walk.l, dQ)], dKs, dVs


@pytest.mark.parametrize("family", [0, 1, 2])
@pytest.mark.parametrize("dtype,spec", CASES, ids=lambda v: v if isinstance(v, str) else "-".join(f"{k}{x}" for k, x in v.items() if k != "chunk_rows"))
def test_walk_calls_equal_the_walk_chunk_by_chunk(dtype, spec, family):
    if family and spec["d"] != 128:
        pytest.skip("the kernel families differ at d = 128 only")
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(dtype=dtype, seed=97, device=DEV, **spec)
        mk = lambda: RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0),
                              case.get("kv_heads", 0))
        want, dKs0, dVs0 = chunk_by_chunk(case, mk())
        walk = mk()
        for t in (walk.O_acc, walk.m, walk.l, walk.O, walk.lse, walk.D):
            t.fill_(float("nan"))                   # nothing of the buffers' contents may get into a fresh walk
        O, lse = walk.forward(case["K"], case["V"], case["k_offs"], masks=case.get("masks"))
        dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
        torch.cuda.synchronize()
        if dtype == "bf16" and spec["d"] != 20 and sum(spec["chunk_rows"]) < 1280:    # (fp32 kernels, split keys: another order of sums)
            for name, a, b in zip(("O", "lse", "O_acc", "m", "l", "dQ"), (O, lse, walk.O_acc, walk.m, walk.l, dQ), want):
                assert torch.equal(a, b), name
            for a, b in zip(dKs + dVs, dKs0 + dVs0):
                assert torch.equal(a, b)
        else:                                       # fp32 sums of at most 2100 terms in another order; bf16 O may round the other way
            assert torch.allclose(lse, want[1], rtol=0, atol=1e-5)
            assert torch.allclose(O.float(), want[0].float(), rtol=2 ** -7 if dtype == "bf16" else 1e-5, atol=1e-3 if dtype == "bf16" else 1e-5)
            for a, b in zip([dQ] + dKs + dVs, [want[5]] + dKs0 + dVs0):   # (bf16: D comes from that O)
                assert float((a - b).norm()) <= (2e-3 if dtype == "bf16" else 1e-5) * float(b.norm())
        compare_all_heads(case, dtype, O, lse, dQ, dKs, dVs)
        # the same gradients in the inputs' type: each fp32 value rounded once
        hQ, hKs, hVs = walk.backward_in_dtype(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
        torch.cuda.synchronize()
        for a, b in zip([hQ, *hKs, *hVs], [dQ, *dKs, *dVs]):
            assert a.dtype == case["Q"].dtype and torch.equal(a, b.to(a.dtype))
    finally:
        B.burst_set_kernel_family(0)


def in_three_layouts(case):
    """The chunks head-major, sequence-major, packed, packed and head-major."""
    def lay(t, how):
        rows = t.transpose(1, 2).contiguous()       # [B, rows, H, d]
        return t if how == 0 else rows.transpose(1, 2) if how == 1 else torch.cat([rows, rows], 2)[:, :, :2].transpose(1, 2)

    for name in ("K", "V"):
        case[name] = [lay(t, how) for t, how in zip(case[name], (0, 1, 2, 2, 0))]


@pytest.mark.parametrize("family", [1, 2])
def test_chunks_of_different_pitch_in_one_walk(family):
    """Head-major, sequence-major and packed chunks in turn, d = 128: the hand-scheduled kernels take one row pitch a launch."""
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(B=2, H=2, d=128, Nq=257, chunk_rows=[100, 64, 190, 128, 65], dtype="bf16", seed=101, device=DEV,
                                   causal=True, q_off=290)

        in_three_layouts(case)
        assert len({k.stride(2) for k in case["K"]}) == 3
        mk = lambda: RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"])
        want, dKs0, dVs0 = chunk_by_chunk(case, mk())
        walk = mk()
        O, lse = walk.forward(case["K"], case["V"], case["k_offs"])
        dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"])
        torch.cuda.synchronize()
        for a, b in zip((O, lse, walk.O_acc, walk.m, walk.l, dQ, *dKs, *dVs), (*want, *dKs0, *dVs0)):
            assert torch.equal(a, b)
        compare_all_heads(case, "bf16", O, lse, dQ, dKs, dVs)
    finally:
        B.burst_set_kernel_family(0)


@pytest.mark.parametrize("d", [4, 32, 64, 96, 128])
@pytest.mark.parametrize("rows", [100, 257])
def test_fp32_chunks_of_different_pitch_in_one_walk(d, rows):
    """The same in fp32, whose kernels go from one pitch to the next inside a launch: dealt to several workgroups per block
    (with a workspace) and not; fp32 sums in another order than chunk by chunk, 1e-5 of the norm."""
    case = workloads.make_case(B=2, H=2, d=d, Nq=rows, chunk_rows=[200, 128, 1100, 256, 130], dtype="f32", seed=107, device=DEV,
                               causal=True, q_off=1557)
    in_three_layouts(case)
    assert len({k.stride(2) for k in case["K"]}) == 3
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"])
    want, dKs0, dVs0 = chunk_by_chunk(case, walk)
    p = walk._walk_params()
    for split in (True, False):
        dQ = torch.full(tuple(walk.Q.shape), float("nan"), device=DEV)
        dKs, dVs = [[torch.full(tuple(k.shape), float("nan"), device=DEV) for k in case["K"]] for _ in range(2)]
        chunks = B.chunk_array(case["K"], case["V"], case["k_offs"], None, p, dKs, dVs, torch.float32)
        need = B.burst_walk_workspace_bytes(chunks, p)
        assert need > 0
        ws = torch.empty(need, device=DEV, dtype=torch.uint8) if split else None
        B.burst_walk_fwd(walk.Q, chunks, walk.O_acc, walk.m, walk.l, walk.O, walk.lse, p, ws)
        B.burst_walk_bwd(walk.Q, chunks, walk.O, case["dO"], walk.lse, walk.D, dQ, p, accumulate_dq=False, workspace=ws)
        torch.cuda.synchronize()
        assert torch.allclose(walk.lse, want[1], rtol=0, atol=1e-5)
        for a, b in zip([walk.O, dQ, *dKs, *dVs], [want[0], want[5], *dKs0, *dVs0]):
            assert float((a - b).norm()) <= 1e-5 * float(b.norm())
        compare_all_heads(case, "f32", walk.O, walk.lse, dQ, dKs, dVs)


@pytest.mark.parametrize("spec,family", [
    (dict(d=64, Nq=70, chunk_rows=[20] * 37, causal=True, q_off=700), 0),
    (dict(d=20, Nq=70, chunk_rows=[20] * 37, causal=True, q_off=700), 0),
    (dict(d=127, Nq=37, chunk_rows=[20] * 37, causal=True, q_off=700), 0),      # dQ: a multiple of 4 elements and two more
    (dict(H=1, d=3, Nq=1, chunk_rows=[20] * 37), 0),                            # three elements
    (dict(H=1, d=1, Nq=69, chunk_rows=[20] * 37), 0),                           # one more
    (dict(d=128, Nq=300, chunk_rows=[256, 70], block=256, pattern="random", density=0.5), 1),
], ids=["d64-37-chunks", "d20-37-chunks", "d127-37-chunks", "d3-one-row", "d1-37-chunks", "d128-flags"])
def test_differentiable_call_of_several_launches(spec, family):
    """The state between the launches lies in the workspace, as dQ does: the same bits as a walk that keeps it."""
    from paper_2403_09347_amd.autograd import burst_attention
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(B=1, dtype="bf16", seed=103, device=DEV, **dict(dict(H=2), **spec))
        walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], block=case.get("block", 0))
        p = walk._walk_params()
        chunks = B.chunk_array(case["K"], case["V"], case["k_offs"], case.get("masks"), p)
        for flag, floats in ((B.BURST_WALK_NO_STATE, spec["d"] + 2), (B.BURST_WALK_HALF_GRADS, spec["d"])):   # several launches
            assert B.burst_walk_workspace_bytes(chunks, p, flag) >= spec.get("H", 2) * spec["Nq"] * floats * 4
        args = case["K"], case["V"], case["k_offs"]
        O0, lse0 = walk.forward(*args, masks=case.get("masks"))
        dQ, dKs, dVs = walk.backward_in_dtype(*args, case["dO"], masks=case.get("masks"))
        full = walk.backward(*args, case["dO"], masks=case.get("masks"))[0]   # fp32
        assert torch.equal(dQ, full.to(dQ.dtype))
        n = len(case["K"])
        leaves = [t.clone().requires_grad_(True) for t in [case["Q"], *case["K"], *case["V"]]]
        O, lse = burst_attention(leaves[0], leaves[1:n + 1], leaves[n + 1:], causal=case["causal"], q_off=case["q_off"],
                                 block_masks=case.get("masks"), block=case.get("block", 0))
        assert torch.equal(O, O0) and torch.equal(lse, lse0)
        for a, b in zip(torch.autograd.grad(O, leaves, case["dO"]), [dQ, *dKs, *dVs]):
            assert torch.equal(a, b)
    finally:
        B.burst_set_kernel_family(0)


def test_walk_calls_without_a_visible_or_any_chunk():
    case = workloads.make_case(B=1, H=2, d=64, Nq=70, chunk_rows=[40, 33], dtype="bf16", seed=3, device=DEV, causal=True,
                               q_off=0, k_offs=[1000, 2000])
    walk = RingWalk(case["Q"], case["scale"], True, 0)
    for Ks, Vs, offs in ((case["K"], case["V"], case["k_offs"]), ([], [], [])):
        for t in (walk.O_acc, walk.m, walk.l, walk.O, walk.lse):
            t.fill_(3.0)
        O, lse = walk.forward(Ks, Vs, offs)
        dQ, dKs, dVs = walk.backward(Ks, Vs, offs, case["dO"])
        hQ, hKs, hVs = walk.backward_in_dtype(Ks, Vs, offs, case["dO"])
        assert all(torch.all(g == 0) for g in [hQ, *hKs, *hVs])
        kept = torch.full_like(dQ, 2.0)
        walk.backward(Ks, Vs, offs, case["dO"], dQ=kept)
        torch.cuda.synchronize()
        assert torch.all(O == 0) and torch.all(torch.isneginf(lse)) and torch.all(walk.O_acc == 0)
        assert torch.all(walk.l == 0) and torch.all(torch.isneginf(walk.m)) and torch.all(dQ == 0) and torch.all(kept == 2.0)
        assert all(torch.all(g == 0) for g in dKs + dVs)


def test_differentiable_call_partial_gradients_and_errors():
    """The native autograd node: gradients for some inputs only, no gradient at all, views it cannot read in
    place, and the exceptions of bad arguments."""
    from paper_2403_09347_amd.autograd import burst_attention
    case = workloads.make_case(B=1, H=4, kv_heads=2, d=64, Nq=70, chunk_rows=[64, 33], dtype="bf16", seed=5, device=DEV,
                               causal=True, q_off=27)
    q, ks, vs = case["Q"], case["K"], case["V"]
    ref = [t.clone().requires_grad_(True) for t in [q, *ks, *vs]]
    O, lse = burst_attention(ref[0], ref[1:3], ref[3:5], causal=True, q_off=27)
    full = torch.autograd.grad(O, ref, case["dO"])
    for wanted in ([0], [2], [1, 4]):
        some = [t.clone() for t in [q, *ks, *vs]]
        for i in wanted:
            some[i].requires_grad_(True)
        O1, lse1 = burst_attention(some[0], some[1:3], some[3:5], causal=True, q_off=27)
        assert torch.equal(O1, O) and torch.equal(lse1, lse) and not lse1.requires_grad
        for i, g in zip(wanted, torch.autograd.grad(O1, [some[i] for i in wanted], case["dO"])):
            assert torch.equal(g, full[i])
    with torch.no_grad():
        assert not burst_attention(ref[0], ref[1:3], ref[3:5], causal=True, q_off=27)[0].requires_grad
    # rows 130 elements apart start off the 16-byte grid: copied, same results
    wide = torch.zeros((1, 4, 70, 130), device=DEV, dtype=torch.bfloat16)
    wide[..., :64] = q
    O2, _ = burst_attention(wide[..., :64], ks, vs, causal=True, q_off=27)
    assert torch.equal(O2, O)
    with pytest.raises(B.BurstError):
        burst_attention(q, ks, vs, scale=-1.0)
    with pytest.raises(ValueError):
        burst_attention(q, ks, vs, block_masks=[torch.ones((1, 1), device=DEV)] * 2, block=64)
    with pytest.raises(ValueError):
        burst_attention(q, [k.float() for k in ks], vs)


@pytest.mark.parametrize("moved", [{0}, {1, 2}, {3}, {4, 5}])
def test_saved_tensors_come_back_in_another_layout(moved):
    """Hooks on saved tensors may give back dense copies of some of the sequence-major tensors (here by position:
    Q, O, lse, keys, values): the gradients are the same bits."""
    from paper_2403_09347_amd.autograd import burst_attention
    gen = torch.Generator(device=DEV).manual_seed(11)
    draw = lambda n, h: torch.randn((2, n, h, 64), device=DEV, generator=gen).bfloat16().transpose(1, 2).requires_grad_(True)
    q, ks, vs, dO = draw(70, 4), [draw(64, 2), draw(33, 2)], [draw(64, 2), draw(33, 2)], draw(70, 4).detach()
    O, _ = burst_attention(q, ks, vs, causal=True, q_off=27)
    want = torch.autograd.grad(O, [q, *ks, *vs], dO)
    packed = []

    def pack(t):
        packed.append(t)
        return t.detach().contiguous() if len(packed) - 1 in moved else t.detach()

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):
        O, _ = burst_attention(q, ks, vs, causal=True, q_off=27)
    assert len(packed) >= 7
    for a, b in zip(torch.autograd.grad(O, [q, *ks, *vs], dO), want):
        assert torch.equal(a, b)


def test_captured_walk_outlives_the_workspace_of_a_longer_one():
    """A captured walk that splits its keys, replayed after the same object has walked more chunks eagerly
    (a larger workspace): every replay equals the eager walk and writes nothing that others own."""
    case = workloads.make_case(B=1, H=2, d=64, Nq=40, chunk_rows=[1024] * 6, dtype="bf16", seed=9, device=DEV)
    walk = RingWalk(case["Q"], case["scale"])
    args = case["K"][:2], case["V"][:2], case["k_offs"][:2]

    def both():
        O, lse = walk.forward(*args)
        return [O, lse, *walk.backward(*args, case["dO"])[:1]]

    want = [t.clone() for t in both()]
    held = walk._workspace.numel()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        both()
    torch.cuda.current_stream().wait_stream(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = both()
    for _ in range(3):
        walk.forward(case["K"], case["V"], case["k_offs"])
        assert walk._workspace.numel() > held
        others = [torch.full((held,), 7, device=DEV, dtype=torch.uint8) for _ in range(4)]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert all(bool((t == 7).all()) for t in others)


def test_differentiable_call_with_flags_for_some_chunks_only():
    """block_masks may hold None for a chunk without flags: the same O, lse and gradients as the walk gives."""
    from paper_2403_09347_amd.autograd import burst_attention
    case = workloads.make_case(B=1, H=2, d=64, Nq=100, chunk_rows=[90, 70, 64], dtype="bf16", seed=13, device=DEV, block=64,
                               pattern="random", density=0.5)
    for masks in ([case["masks"][0], None, case["masks"][2]], [None, case["masks"][1], None], [None] * 3):
        walk = RingWalk(case["Q"], case["scale"], block=64)
        O0, lse0 = walk.forward(case["K"], case["V"], case["k_offs"], masks=masks)
        dQ, dKs, dVs = walk.backward_in_dtype(case["K"], case["V"], case["k_offs"], case["dO"], masks=masks)
        leaves = [t.clone().requires_grad_(True) for t in [case["Q"], *case["K"], *case["V"]]]
        O, lse = burst_attention(leaves[0], leaves[1:4], leaves[4:], block_masks=masks, block=64)
        assert torch.equal(O, O0) and torch.equal(lse, lse0)
        for a, b in zip(torch.autograd.grad(O, leaves, case["dO"]), [dQ, *dKs, *dVs]):
            assert torch.equal(a, b)


def test_workspace_belongs_to_the_stream_that_uses_it(monkeypatch):
    """One walk object on two streams in turn, shorter and longer walks: every workspace handed to the library was
    allocated on the stream of that call, so that the allocator cannot give it away while the call's kernels run."""
    case = workloads.make_case(B=1, H=2, d=64, Nq=40, chunk_rows=[1024] * 6, dtype="bf16", seed=9, device=DEV)
    walk = RingWalk(case["Q"], case["scale"])
    used, real = [], B.burst_walk_fwd

    def spy(*args):
        ws = args[-1]
        at = [s["stream"] for s in torch.cuda.memory_snapshot() if s["address"] <= ws.data_ptr() < s["address"] + s["total_size"]]
        used.append((at, torch.cuda.current_stream().cuda_stream))
        real(*args)

    monkeypatch.setattr(B, "burst_walk_fwd", spy)
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    outs = []
    for stream, n in ((main, 2), (side, 2), (side, 4), (main, 6), (side, 6)):
        stream.wait_stream(main if stream is side else side)
        with torch.cuda.stream(stream):
            outs.append([t.clone() for t in walk.forward(case["K"][:n], case["V"][:n], case["k_offs"][:n])])
    torch.cuda.synchronize()
    assert len(used) == 5 and all(at == [now] for at, now in used)
    for i, j in ((0, 1), (3, 4)):
        assert all(torch.equal(a, b) for a, b in zip(outs[i], outs[j]))

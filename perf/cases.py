"""The work that users of this package have it do, as cases that can be timed: one device's share of a
sequence-parallel ring (forward walk over key/value chunks, then the backward walk), differentiable
attention calls inside a training step, and forward-only calls of a few new rows against resident keys.

A case is a dict of plain values:
  kind    "walk"      harness.RingWalk: forward over all chunks, then backward over all chunks
          "ring"      harness.DoubleBufferedWalk: the same with every chunk copied from a source pool
                      into one of two receive buffers while the chunk before it is computed
          "autograd"  autograd.burst_attention and the gradients of its inputs
          "forward"   harness.RingWalk, the forward walk only
  dtype, B, H, KV (key/value heads), d, Nq, G (chunks), Nc (rows of a chunk), causal, q_off, window,
  block (edge of block-sparse flags, 0 = none), density (share of flags set), layout ("head": dense
  [B, H, rows, d]; "seq": views of [B, rows, H, d] tensors).
Inputs are N(0, 1), as everywhere in this repository (activations of a normalised layer)."""
import math

import numpy as np
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.autograd import burst_attention
from paper_2403_09347_amd.harness import DoubleBufferedWalk, RingWalk


def _case(kind, dtype="bf16", B=1, H=32, KV=0, d=128, Nq=4096, G=8, Nc=4096, causal=False, q_off=0, window=0,
          block=0, density=0.0, layout="head", name=None):
    c = dict(kind=kind, dtype=dtype, B=B, H=H, KV=KV or H, d=d, Nq=Nq, G=G, Nc=Nc, causal=causal, q_off=q_off,
             window=window, block=block, density=density, layout=layout)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The benchmark's smallest configuration: one fp32 head, four chunks of 256 rows.  Checks of a
        # port or of a new ring schedule run at this size, thousands of times.
        _case("walk", "f32", H=1, d=64, Nq=256, G=4, Nc=256, name="f32_tiny_ring"),
        # fp32 attention where bf16 will not do (references, fine-tuning of small layers), ragged sizes.
        _case("walk", "f32", H=8, d=128, Nq=700, G=2, Nc=700, causal=True, q_off=700, name="f32_causal_ragged"),
        # The benchmark's headline: one device's share of 32 heads, 32K tokens on 8 devices.
        _case("walk", name="llama7b_32k_G8"),
        # The same ring as it runs with transfers: last rank of a causal sequence, chunks arriving
        # through the double buffer.
        _case("ring", causal=True, q_off=7 * 4096, name="ring_last_rank_causal"),
        # Long slices (40 heads, 16K rows a device): two block pairs of the 128K / 8 configuration.
        _case("walk", H=40, Nq=16384, G=2, Nc=16384, name="llama13b_16k_pairs"),
        # A short sequence over many devices: 512 rows a device, the launch-bound end of a causal ring.
        _case("walk", Nq=512, G=16, Nc=512, causal=True, q_off=15 * 512, name="short_slices_causal"),
        # Training step of a layer with 64-wide heads: causal self-attention of a batch of short texts.
        _case("autograd", B=4, H=16, d=64, Nq=1024, G=1, Nc=1024, causal=True, name="d64_self_attention"),
        # Grouped heads, sequence-major activations as a projection leaves them, and a length that is no
        # multiple of anything.
        _case("autograd", KV=8, Nq=3001, G=1, Nc=3001, causal=True, layout="seq", name="grouped_ragged_seq"),
        # Heads that are neither 64 nor 128 wide.
        _case("autograd", B=2, H=16, d=96, Nq=777, G=1, Nc=777, causal=True, name="d96_self_attention"),
        # Sliding window over a long context, last rank of the ring.
        _case("walk", causal=True, q_off=7 * 4096, window=4096, name="window_last_rank"),
        # Block-sparse attention with 64-wide blocks, a quarter of them set.
        _case("walk", G=2, block=64, density=0.25, name="block64_quarter"),
        # A few new rows against a long resident context (scoring a continuation), forward only.
        _case("forward", Nq=40, G=8, Nc=4096, causal=True, q_off=8 * 4096 - 40, name="few_rows_long_context"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rows(rng, lo, hi):
    """Rows over the whole range: half of the draws a multiple of 64, the others as they come."""
    n = _log(rng, lo, hi)
    return max(64, n // 64 * 64) if rng.random() < 0.5 else n


# What a drawn case may cost, in multiply-adds times two of the visible pairs (the largest listed
# case has 3.8e13): matrix-core shapes, and those that have none at present.
_MOST = {"bf16": 1.2e13, "f32": 1.5e11}


def draw(rng):
    while True:
        kind = rng.choice(["walk", "walk", "walk", "ring", "autograd", "autograd", "forward"])
        c = _case(kind)
        if kind in ("walk", "ring"):
            if kind == "walk" and rng.random() < 0.25:
                c.update(dtype="f32", H=rng.choice([1, 2, 4, 8]), d=rng.choice([32, 40, 64, 80, 128]),
                         Nq=_rows(rng, 100, 1500), G=rng.choice([1, 2, 3, 4]))
                c.update(Nc=c["Nq"] if rng.random() < 0.7 else _rows(rng, 100, 1500))
            else:
                c.update(H=rng.choice([8, 12, 16, 32, 40]), d=rng.choice([128, 128, 128, 64]),
                         Nq=_rows(rng, 256, 16384), G=rng.choice([1, 2, 3, 4, 6, 8, 12, 16]))
                c.update(Nc=c["Nq"] if rng.random() < 0.8 else _rows(rng, 256, 16384))
            c["KV"] = c["H"]
            if rng.random() < 0.6:
                c.update(causal=True, q_off=max(0, rng.randrange(c["G"]) * c["Nc"]))
                if rng.random() < 0.3:
                    c["window"] = _log(rng, 128, 8192)
            if kind == "walk" and c["dtype"] == "bf16" and not c["window"] and rng.random() < 0.25:
                c.update(block=rng.choice([64, 128, 256]), density=rng.choice([0.1, 0.25, 0.5]))
        elif kind == "autograd":
            n = _rows(rng, 128, 8192)
            c.update(B=rng.choice([1, 1, 2, 4]), H=rng.choice([8, 16, 32]), d=rng.choice([64, 64, 80, 96, 128, 128]),
                     Nq=n, G=1, Nc=n, causal=rng.random() < 0.75, layout=rng.choice(["head", "seq"]))
            c["KV"] = c["H"] // rng.choice([1, 1, 4])
        else:
            c.update(B=rng.choice([1, 2, 4]), H=rng.choice([8, 32, 40]), d=rng.choice([64, 128, 128]),
                     Nq=_log(rng, 1, 200), G=rng.choice([1, 2, 4, 8]), Nc=_rows(rng, 256, 8192), causal=True)
            c["q_off"] = max(0, c["G"] * c["Nc"] - c["Nq"])
            c["KV"] = c["H"] // rng.choice([1, 1, 4])
        tiled = c["dtype"] == "bf16" and c["d"] in (64, 128) and (c["KV"] == c["H"] or c["Nq"] % 64 == 0)
        most = _MOST["bf16" if tiled else "f32"]
        if 1e8 < work(c)["flops"] < most and _rows_walked(c) < 40 * 32768 * 4:
            return c


def _rows_walked(c):
    return c["B"] * c["H"] * (c["Nq"] + c["G"] * c["Nc"])


def _visible_pairs(c):
    """(query, key) pairs of one head that the masks leave (block flags: the expected number)."""
    nk = c["G"] * c["Nc"]
    if c["causal"] or c["window"]:
        pos = c["q_off"] + np.arange(c["Nq"], dtype=np.int64)
        hi = np.minimum(nk, pos + 1) if c["causal"] else np.full_like(pos, nk)
        lo = np.maximum(0, pos - c["window"] + 1) if c["window"] else np.zeros_like(pos)
        pairs = float(np.maximum(0, hi - lo).sum())
    else:
        pairs = float(c["Nq"]) * nk
    return pairs * (c["density"] if c["block"] else 1.0)


def work(case):
    """Every input read once, every output written once; 4 d operations per visible pair forward, 10 d
    backward.  Gradients are fp32 from a walk and of the input type from autograd."""
    e = 2 if case["dtype"] == "bf16" else 4
    q = case["B"] * case["H"] * case["Nq"]
    kv = 2 * case["B"] * case["KV"] * case["G"] * case["Nc"]
    pairs = case["B"] * case["H"] * _visible_pairs(case)
    nbytes = (2 * q + kv) * case["d"] * e + 4 * q                     # Q, K, V in, O and lse out
    flops = 4.0 * case["d"] * pairs
    if case["kind"] != "forward":
        g = e if case["kind"] == "autograd" else 4
        nbytes += q * case["d"] * e + (q + kv) * case["d"] * g        # dO in, dQ, dK, dV out
        flops += 10.0 * case["d"] * pairs
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    # Measured against the same arithmetic in 64 bits on the stored inputs, the largest figure of any
    # output over these ranges: bf16 0.0025 (P, dS and O are rounded to bf16, 2^-9 each; the largest
    # single difference, 0.14 of the root mean square, belongs to gradients of causal rows that see a
    # handful of keys), fp32 7.7e-7 (largest single difference 1.0e-5).  About four times each.
    return {"rel": 0.01, "max": 0.5} if case["dtype"] == "bf16" else {"rel": 3.5e-6, "max": 5e-5}


def prepare(case, seed):
    c = case
    n = workloads.make_case(B=c["B"], H=c["H"], d=c["d"], Nq=c["Nq"], chunk_rows=[c["Nc"]] * c["G"], dtype=c["dtype"],
                            seed=seed, device="cuda", causal=c["causal"], q_off=c["q_off"], window=c["window"],
                            block=c["block"], pattern="random", density=c["density"] or 0.4,
                            kv_heads=c["KV"] if c["KV"] != c["H"] else 0, layout=c["layout"])
    s = dict(n, kind=c["kind"], masks=n.get("masks"))
    if c["kind"] == "autograd":
        s["leaves"] = [t.requires_grad_(True) for t in [n["Q"]] + n["K"] + n["V"]]
    elif c["kind"] == "ring":
        s["walk"] = DoubleBufferedWalk(n["Q"], n["scale"], n["causal"], n["q_off"], c["Nc"], n["window"])
    else:
        s["walk"] = RingWalk(n["Q"], n["scale"], n["causal"], n["q_off"], n["window"], c["block"], n.get("kv_heads", 0))
    return s


def run(state):
    s = state
    if s["kind"] == "autograd":
        O, lse = burst_attention(s["Q"], s["K"], s["V"], s["scale"], s["causal"], s["q_off"], s["window"])
        return [O, lse, *torch.autograd.grad(O, s["leaves"], s["dO"])]
    walk = s["walk"]
    if s["kind"] == "ring":
        O, lse = walk.forward(s["K"], s["V"], s["k_offs"])
        dQ, dKs, dVs = walk.backward(s["K"], s["V"], s["k_offs"], s["dO"])
        return [O, lse, dQ, *dKs, *dVs]
    O, lse = walk.forward(s["K"], s["V"], s["k_offs"], masks=s["masks"])
    if s["kind"] == "forward":
        return [O, lse]
    dQ, dKs, dVs = walk.backward(s["K"], s["V"], s["k_offs"], s["dO"], masks=s["masks"])
    return [O, lse, dQ, *dKs, *dVs]

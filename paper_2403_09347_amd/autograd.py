"""Attention of a query slice against a list of key/value chunks (paper Alg. 1 for the forward, Alg. 2 for
the backward) as one differentiable torch call.  The autograd node is native (csrc/burst_torch.cpp):
argument marshalling and buffer management, every arithmetic step a library call.  On one GPU the
chunks are simply all resident; in a ring the same calls are made once per received chunk."""
import torch

from . import binding as B


def burst_attention(q, k_chunks, v_chunks, scale=None, causal=False, q_off=0, window=0, block_masks=None, block=0):
    """q [B, H, Nq, d]; k_chunks / v_chunks: lists of [B, Hkv, Nc_j, d] (Hkv divides H), chunk j
    starting at global key position sum(Nc_0..Nc_{j-1}); q_off = global position of query row 0.
    Returns (O [B, H, Nq, d] in q's dtype and memory layout, lse [B, H, Nq] fp32).  Gradients flow
    to q and to every chunk (rounded to the input dtype).  Views with a contiguous last dimension
    (sequence-major tensors, slices of a packed projection) are read in place, without a copy.
    block_masks: one uint8 device tensor of block flags per chunk (see binding.params) with blocks
    of `block` rows / keys, or None for a chunk without flags; or None.
    Results are the same bits whenever a call is repeated; the order of the fp32 sums, and with it the last bits, depends on all
    sizes of a call, the number of heads among them.
    The node saves its inputs, O and lse as torch's own operations do: a tensor changed in place before the backward is
    an error, and a second backward needs retain_graph."""
    if isinstance(k_chunks, torch.Tensor):
        k_chunks, v_chunks = [k_chunks], [v_chunks]
    assert len(k_chunks) == len(v_chunks) and len(k_chunks) > 0
    scale = float(scale) if scale is not None else q.shape[-1] ** -0.5
    if block_masks is not None:
        assert len(block_masks) == len(k_chunks) and block > 0
    try:
        O, lse = B.load_torch_module().attention(q, list(k_chunks), list(v_chunks), [] if block_masks is None else list(block_masks),
                                                 scale, bool(causal), int(q_off), int(window),
                                                 0 if block_masks is None else int(block))
    except RuntimeError as e:
        raise B.from_native(e) from None
    return O, lse

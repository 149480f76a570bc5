"""Causal grids with more than one and at most two workgroups per CU (their second half is mirrored): every head
must get the bits it gets in a call of a few heads, at the edges of the rule and off the multiples of 8."""
import pytest
import torch

from paper_2403_09347_amd.autograd import burst_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,N,d", [(256, 100, 64), (257, 100, 64), (129, 130, 64), (85, 700, 64), (171, 257, 64), (128, 512, 64),
                                   (60, 600, 96), (100, 321, 80), (90, 385, 32)])
def test_every_head_as_in_a_small_call(H, N, d):
    gen = torch.Generator(device="cuda:0").manual_seed(H)
    q, k, v, dO = [torch.randn((1, H, N, d), device="cuda:0", generator=gen).bfloat16() for _ in range(4)]

    def call(a, b):
        x = [t[:, a:b].clone().requires_grad_(True) for t in (q, k, v)]
        O, lse = burst_attention(*x, causal=True)
        return [O.detach(), lse, *torch.autograd.grad(O, x, dO[:, a:b])]

    whole = call(0, H)
    parts = [call(a, min(a + 16, H)) for a in range(0, H, 16)]
    for i, t in enumerate(whole):
        assert torch.equal(t, torch.cat([p[i] for p in parts], dim=1))

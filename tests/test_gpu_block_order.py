"""Causal grids whose workgroups are taken by block instead of head by head: every head must get the bits it gets in a call
of a few heads, with numbers of heads that are and are not multiples of 8, in the hand-scheduled, the plain and the fp32
kernels, forward, dQ and dK/dV, and where a head is long enough to be taken whole again; and, shorter ones, the oracle's values."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd.autograd import burst_attention
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,N,d,dtype,family,few", [
    (68, 777, 128, torch.bfloat16, 1, 17), (72, 777, 128, torch.bfloat16, 1, 8), (110, 300, 128, torch.bfloat16, 2, 11),
    (18, 1000, 32, torch.float32, 0, 9), (22, 900, 128, torch.float32, 0, 11), (16, 2100, 8, torch.float32, 0, 8),
    (76, 900, 64, torch.bfloat16, 0, 19), (16, 17000, 8, torch.bfloat16, 0, 8),
])
def test_every_head_as_in_a_small_call(H, N, d, dtype, family, few):
    assert few < H                                   # (else the parts are the call itself)
    gen = torch.Generator(device="cuda:0").manual_seed(H)
    q, k, v, dO = [torch.randn((1, H, N, d), device="cuda:0", generator=gen).to(dtype) for _ in range(4)]

    def call(a, b):
        x = [t[:, a:b].clone().requires_grad_(True) for t in (q, k, v)]
        O, lse = burst_attention(*x, causal=True)
        return [O.detach(), lse, *torch.autograd.grad(O, x, dO[:, a:b])]

    B.burst_set_kernel_family(family)
    try:
        whole = call(0, H)
        again = call(0, H)
        parts = [call(a, min(a + few, H)) for a in range(0, H, few)]
    finally:
        B.burst_set_kernel_family(0)
    for i, t in enumerate(whole):
        assert torch.isfinite(t.float()).all()
        assert torch.equal(t, again[i])
        assert torch.equal(t, torch.cat([p[i] for p in parts], dim=1))
    if N <= 2100:
        case = dict(Q=q, K=[k], V=[v], dO=dO, k_offs=[0], scale=d ** -0.5, causal=True, q_off=0)
        compare_all_heads(case, "f32" if dtype == torch.float32 else "bf16", *whole[:3], [whole[3]], [whole[4]], heads=[0, H // 2, H - 1],
                          dkv_kind="rel")

"""Infinities and NaN in the inputs of the calls that the scalar kernels once had (fp32, bf16 head dimensions other than 64
and 128, dK and dV of grouped heads whose slice is no multiple of 64 rows): every output is infinite or NaN exactly
where the formula makes it so over the pairs that are visible, and right everywhere else.  Matrix products multiply more
than these pairs (hidden ones, the zeros of padding, the lower parts of a probability), see csrc/burst_rows.h."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import TOL, f64, head_inputs, pattern_of

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")

SPECS = [
    ("bf16", dict(H=2, d=96, Nq=130, chunk_rows=[100, 70])),
    ("bf16", dict(H=2, d=40, Nq=130, chunk_rows=[100, 70], causal=True, q_off=40)),
    ("bf16", dict(H=2, d=72, Nq=130, chunk_rows=[100, 130], causal=True, q_off=100, window=60)),
    ("bf16", dict(H=2, d=80, Nq=100, chunk_rows=[90, 70], block=64, pattern="random", density=0.5)),
    ("bf16", dict(H=2, d=96, Nq=33, chunk_rows=[800, 700], causal=True, q_off=1467)),     # split keys
    ("bf16", dict(H=2, d=20, Nq=70, chunk_rows=[40, 33], causal=True, q_off=3)),
    ("f32", dict(H=2, d=64, Nq=100, chunk_rows=[90, 70])),
    ("f32", dict(H=2, d=128, Nq=130, chunk_rows=[100, 70], causal=True, q_off=40)),
    ("f32", dict(H=2, d=40, Nq=100, chunk_rows=[90, 70], block=64, pattern="random", density=0.5)),
    ("f32", dict(H=4, kv_heads=2, d=34, Nq=70, chunk_rows=[40, 33], causal=True, q_off=3)),
]
GROUPED = ("bf16", dict(H=4, kv_heads=2, d=128, Nq=100, chunk_rows=[90, 70], causal=True, q_off=60))


def plant(case, what):
    Q, K, V, dO = case["Q"], case["K"], case["V"], case["dO"]
    if what == "V inf":
        V[0][:, :, 5, 3] = INF
        V[1][:, :, 7, 3] = -INF
        V[1][:, :, -1, -1] = INF
    elif what == "V NaN in the last keys":
        V[1][:, :, -10:] = NAN
    elif what == "scores -inf":                     # column 0 of Q is positive
        Q[..., 0] = Q[..., 0].abs() + 0.1
        K[0][:, :, 5:9, 0] = -INF
        K[1][:, :, 32:, 0] = -INF
    elif what == "scores -inf, last column":
        Q[..., -1] = Q[..., -1].abs() + 0.1
        K[0][:, :, 5:9, -1] = -INF
        K[1][:, :, -1, -1] = -INF
    elif what == "all scores -inf":
        Q[..., 0] = Q[..., 0].abs() + 0.1
        for k in K:
            k[..., 0] = -INF
    elif what == "dO inf":
        dO[:, :, 11, 3] = INF
        dO[:, :, 30, 1] = -INF
    else:
        assert what == "dO NaN"
        dO[:, :, 11, 3] = NAN


def product(W, X, seen):
    """W X over the seen pairs only (0 x inf of an unseen pair is nothing)."""
    with np.errstate(invalid="ignore"):
        return np.where(seen[:, :, None], W[:, :, None] * X[None], 0.0).sum(1)


def same(got, want, dtype, name):
    got = f64(got)
    for cls in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(cls(got), cls(want)), (name, cls.__name__, int(cls(got).sum()), int(cls(want).sum()))
    fin = np.isfinite(want)
    if fin.any():
        bar = max(TOL[dtype]["abs"], TOL[dtype]["rel"] * np.abs(want[fin]).max())
        assert np.abs(got[fin] - want[fin]).max() <= bar, name


def check(dtype, spec, what, forward=True):
    case = workloads.make_case(B=1, dtype=dtype, seed=139, device="cuda:0", **spec)
    plant(case, what)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0), case.get("kv_heads", 0))
    args = case["K"], case["V"], case["k_offs"]
    O, lse = walk.forward(*args, masks=case.get("masks"))
    dQ, dKs, dVs = walk.backward(*args, case["dO"], masks=case.get("masks"))
    hQ, hKs, hVs = walk.backward_in_dtype(*args, case["dO"], masks=case.get("masks"))
    into = [torch.ones_like(dQ)] + [[torch.full_like(g, 7.0) for g in gs] for gs in (dKs, dVs)]
    walk.backward(*args, case["dO"], *into, masks=case.get("masks"))
    torch.cuda.synchronize()
    group = spec["H"] // spec.get("kv_heads", spec["H"])
    dK_sum = dV_sum = None
    for h in range(spec["H"]):
        Q, K, V, dO, qp, kp = head_inputs(case, 0, h)
        seen = np.ones((len(qp), len(kp)), bool)
        if case["causal"]:
            seen &= kp[None] <= qp[:, None]
        if case["window"]:
            seen &= kp[None] > qp[:, None] - case["window"]
        pat = pattern_of(case, h=h)
        if pat is not None:
            seen &= pat
        with np.errstate(invalid="ignore", divide="ignore"):
            S = np.where(seen, case["scale"] * product(Q, K.T, np.ones(Q.shape, bool)), -np.inf)
            top = S.max(1)
            none = ~np.isfinite(top)                # no key with a finite score: like a row that sees none
            P = np.exp(S - np.where(none, 0.0, top)[:, None])
            l = P.sum(1)
            P /= np.where(none, 1.0, l)[:, None]
            lse_ref = np.where(none, -np.inf, top + np.log(l))
            O_ref = np.where(none[:, None], 0.0, product(P, V, seen))
            if forward:
                same(lse[0, h], lse_ref, dtype, "lse")
                same(O[0, h], O_ref, dtype, "O")
            D = (dO * f64(O[0, h])).sum(1)
            with_row = seen & ~none[:, None]
            dS = np.where(with_row, P * (product(dO, V.T, np.ones(dO.shape, bool)) - D[:, None]), 0.0)
            dK, dV = case["scale"] * product(dS.T, Q, with_row.T), product(P.T, dO, with_row.T)
            if forward:
                want = case["scale"] * product(dS, K, with_row)
                same(dQ[0, h], want, dtype, "dQ")
                same(into[0][0, h] - 1.0, want, dtype, "dQ added")
                same(hQ[0, h], want, "bf16", "dQ in the inputs' type")
            dK_sum, dV_sum = (dK, dV) if h % group == 0 else (dK_sum + dK, dV_sum + dV)
        if h % group == group - 1:
            for gs, halves, overwritten, want in ((dKs, hKs, into[1], dK_sum), (dVs, hVs, into[2], dV_sum)):
                cat = lambda x: torch.cat([g[0, h // group] for g in x])
                same(cat(gs), want, dtype, "dK, dV")
                same(cat(overwritten), want, dtype, "dK, dV over what was there")
                same(cat(halves), want, "bf16", "dK, dV in the inputs' type")


@pytest.mark.parametrize("what", ["V inf", "V NaN in the last keys", "scores -inf", "scores -inf, last column", "all scores -inf", "dO inf",
                                  "dO NaN"])
@pytest.mark.parametrize("dtype,spec", SPECS, ids=lambda v: v if isinstance(v, str) else "-".join(f"{k}{x}" for k, x in v.items() if k != "chunk_rows"))
def test_infinities_and_nan_stay_where_the_formula_puts_them(dtype, spec, what):
    check(dtype, spec, what)


@pytest.mark.parametrize("what", ["scores -inf", "dO inf", "dO NaN"])
def test_grouped_dkv_with_partial_last_tiles(what):
    """(O and lse come from kernels that multiply hidden pairs too: only their outputs go into the reference.)"""
    check(*GROUPED, what, forward=False)


@pytest.mark.parametrize("dtype,spec", [("bf16", dict(H=2, d=96, Nq=33, chunk_rows=[70, 1, 129])), ("f32", dict(H=2, d=40, Nq=33, chunk_rows=[70, 1, 129])),
                                        ("bf16", dict(H=4, kv_heads=2, d=128, Nq=33, chunk_rows=[70, 1, 129]))],
                         ids=["padded", "f32", "grouped"])
def test_nothing_is_written_past_the_gradients(dtype, spec):
    """Wavefronts past the last key or row see NaN too (padding x infinity) and have nothing to write."""
    case = workloads.make_case(B=1, dtype=dtype, seed=149, device="cuda:0", **spec)
    case["dO"].fill_(NAN)
    walk = RingWalk(case["Q"], case["scale"], kv_heads=case.get("kv_heads", 0))
    walk.forward(case["K"], case["V"], case["k_offs"])
    guard = 16384
    flat = {}

    def inside(name, shape):
        n = int(np.prod(shape))
        flat[name] = torch.full((n + 2 * guard,), 7.0, device="cuda:0")
        return flat[name][guard:guard + n].view(shape)

    dQ = inside("dQ", tuple(case["Q"].shape))
    dKs = [inside(f"dK{j}", tuple(k.shape)) for j, k in enumerate(case["K"])]
    dVs = [inside(f"dV{j}", tuple(k.shape)) for j, k in enumerate(case["K"])]
    walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], dQ, dKs, dVs)
    torch.cuda.synchronize()
    for name, t in flat.items():
        assert bool((t[:guard] == 7.0).all()) and bool((t[-guard:] == 7.0).all()), name
        assert bool(torch.isnan(t[guard:-guard]).all()), name

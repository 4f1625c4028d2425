"""hilore_grpo_coeffs where a workgroup owns two runs of 1024 slots (2^20 slots and
more) and where expm1 leaves its polynomial.

A batch of whole groups is computed at once and in slices below the limit; every
per-slot output of the large call must equal the slices' bit for bit (with N
given, since a slice counts its own).
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def call(hl, rew, new, old, ref, mask, P, G, T, n_norm):
    n = P * G * T
    o = {"adv": torch.full((P * G,), float("nan"), device="cuda"),
         "ratio": torch.full((n,), float("nan"), device="cuda"),
         "flags": torch.full((n,), 0xEE, dtype=torch.uint8, device="cuda"),
         "coeff": torch.full((n,), float("nan"), device="cuda")}
    hl.hilore_grpo_coeffs(rew, new, old, ref, mask, P, G, T, 0.2, 1e-6, 1e-3 if ref is not None else 0.0,
                          n_norm, o["adv"], o["ratio"], o["flags"], o["coeff"])
    return o


@pytest.mark.parametrize("P,G,T", [
    (64, 16, 1024),       # 2^20 slots exactly
    (4096, 4, 65),        # responses across threads, a last workgroup of one run and a bit
    (65600, 16, 1),       # one slot per response: every slot of a thread another response
    (8, 5, 26217),        # runs inside one response, odd total
    (1025, 32, 1025),     # operands past twice the cache: one run again, odd total
])
def test_two_runs_match_one(hl, P, G, T):
    g = torch.Generator(device="cuda").manual_seed(P + G + T)
    R, n = P * G, P * G * T
    assert n >= 1 << 20
    rew = (torch.rand(R, generator=g, device="cuda") < 0.5).float()
    old = torch.randn(n, generator=g, device="cuda") * 0.5 - 2
    new = old + 0.2 * torch.randn(n, generator=g, device="cuda")
    # a tenth of the slots drift past the polynomial's range
    ref = old + torch.randn(n, generator=g, device="cuda") * torch.where(
        torch.rand(n, generator=g, device="cuda") < 0.1, 2.0, 0.05)
    mask = (torch.rand(n, generator=g, device="cuda") < 0.7).to(torch.uint8)
    N = float(int(mask.sum()))
    whole = call(hl, rew, new, old, ref, mask, P, G, T, N)
    counted = call(hl, rew, new, old, ref, mask, P, G, T, 0.0)
    for k in whole:
        assert torch.equal(whole[k], counted[k]), k
    step = max(1, (1 << 19) // (G * T))
    for p in range(0, P, step):
        q = min(P, p + step)
        r, t = slice(p * G, q * G), slice(p * G * T, q * G * T)
        part = call(hl, rew[r].clone(), *(x[t].clone() for x in (new, old, ref, mask)), q - p, G, T, N)
        assert torch.equal(part["adv"], whole["adv"][r])
        for k in ("ratio", "flags", "coeff"):
            assert torch.equal(part[k], whole[k][t]), k


def test_expm1_range(hl):
    """beta expm1(ref - new) alone (equal rewards), across the polynomial's range and beyond."""
    n = 1 << 16
    d = torch.linspace(-0.5, 0.5, n, device="cuda")
    d[::97] *= 0.0
    for x in (d, 1.02 * d, 12.0 * d):
        new = torch.zeros(n, device="cuda")
        rew = torch.ones(16, device="cuda")
        out = call(hl, rew, new, new.clone(), x.contiguous(), None, 1, 16, n // 16, 1.0)
        beta = float(torch.tensor(1e-3, dtype=torch.float32))
        want = -beta * torch.expm1(x.double())
        # equal rewards and N = 1: the coefficient is -beta e, rounded once (half an ulp), with
        # e within 0.86 ulp of expm1 where the polynomial forms it and within 1.5 elsewhere
        # (an ulp of a float is at most 2^-23 of it)
        ulps = torch.where(x.abs() <= 0.5, 0.86 + 0.5, 1.5 + 0.5)
        assert bool(((out["coeff"].double() - want).abs() <= ulps * 2.0 ** -23 * want.abs()).all())

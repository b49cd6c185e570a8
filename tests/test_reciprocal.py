"""The reciprocal of the density in the collisions, against a division.

FP32: on a lattice of one row with populations 0, 2 and 4 only, nothing moves and
each node is a collision of its own density, with a momentum along y that is a
power of two.  The step is compared, value for value, with the collision written out
in correctly rounded FP32 operations on the rounded quotient 1 / rho; every
significand of a binade, and the range a density can be in.  FP64: the velocity of a
channel profile of one column is 2 / rho."""
import numpy as np
import pytest
import torch

from paper_2504_14494_amd import lbm


def _round_odd(s, err):
    """The double s = RN(x) of an exact x = s + err, rounded to odd: rounding
    that to FP32 is rounding x."""
    bits = s.view(torch.int64)
    away = ((err > 0) == (s > 0)).to(torch.int64) * 2 - 1
    move = (err != 0) & ((bits & 1) == 0)
    return torch.where(move, bits + away, bits).view(torch.float64)


def _fma(a, b, c):
    """Fused multiply-add of FP32 tensors."""
    p, c = a.double() * b.double(), torch.as_tensor(c).double()   # exact products
    s = p + c
    t = s - p
    return _round_odd(s, (p - (s - t)) + (c - t)).float()


def _collide(rho, inv, half):
    """BGK at rate 1 of g0 = rho - 1, g2 = half, g4 = -half, with 1 / rho = inv."""
    f = lambda x: torch.tensor(np.float32(x), device=rho.device)
    one, four = np.float32(1), np.float32(4)
    A0, A1 = four / np.float32(9), one / np.float32(9)
    B1, D0 = one / np.float32(3), np.float32(2) / np.float32(3)
    D1 = D0 / four
    A5, B5 = (one - A0 - four * A1) / four, (one - np.float32(2) * B1) / four
    D5 = (np.float32(1.5) - D0 - four * D1) / four
    drho = rho - 1
    g = [torch.zeros_like(rho) for _ in range(9)]
    g[0], g[2], g[4] = drho, torch.full_like(rho, half), torch.full_like(rho, -half)
    v = (2 * half) * inv
    vv = v * v
    out = []
    for i in range(9):
        if i == 0:
            geq = _fma(drho, f(A0).expand_as(rho), rho * -(f(D0) * vv))
        else:
            A, B, C, D = (A1, B1, 0.5, D1) if i < 5 else (A5, B5, 0.125, D5)
            if i in (1, 3):
                e = torch.zeros_like(v)
            else:
                e = v
            b = -B if i in (3, 4, 7, 8) else B
            q = _fma(f(b).expand_as(rho), e, e * (f(C) * e))
            geq = _fma(rho, _fma(f(-D).expand_as(rho), vv, q), f(A) * drho)
        out.append((geq - g[i]) + g[i])
    return torch.stack(out)


def _densities(lo, hi, device):
    """Every FP32 rho in [lo, hi) for which rho - 1 is exact."""
    a, b = (int(np.float32(x).view(np.int32)) for x in (lo, hi))
    rho = torch.arange(a, b, dtype=torch.int32, device=device).view(torch.float32)
    return rho[((rho - 1).double() + 1).float() == rho]


def _quotient(rho):
    return (1.0 / rho.double()).float()     # 53 >= 2 x 24 + 2 bits: no double rounding


def _half(rho_scale):
    """A momentum whose square is most of the equilibrium at such densities."""
    return 32.0 * max(rho_scale, 1.0)


@pytest.mark.parametrize("scale", [0.5, 1.0, 2.0, 1024.0, 2.0 ** 19])
def test_the_comparison_sees_one_unit_in_the_last_place(scale):
    rho = _densities(scale, 2 * scale, "cpu")[::4099]
    inv = _quotient(rho)
    off = (inv.view(torch.int32) + 1).view(torch.float32)
    half = _half(scale)
    seen = (_collide(rho, inv, half) != _collide(rho, off, half)).any(0).float().mean()
    assert float(seen) > 0.99, float(seen)


def _check(rho, half):
    n = rho.numel()
    src = torch.zeros(1, 9, n, device="cuda")
    src[0, 0], src[0, 2], src[0, 4] = rho - 1, half, -half
    got = lbm.lbm_step_bgk(src, torch.empty_like(src), 1.0)[0]
    ref = _collide(rho, _quotient(rho), half)
    assert torch.equal(got, ref), f"{int((got != ref).any(0).sum())} of {n}"


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [0.5, 1.0, 2.0])
def test_every_significand_gives_the_division(scale):
    rho = _densities(scale, 2 * scale, "cuda")
    assert rho.numel() == 1 << 23
    for part in rho.split(1 << 21):
        _check(part, _half(scale))


@pytest.mark.gpu
def test_the_range_of_densities_gives_the_division():
    for k in range(-20, 20):
        rho = _densities(2.0 ** k, 2.0 ** (k + 1), "cuda")
        ends = torch.cat([rho[:2048], rho[-2048:], rho[::997]])
        _check(ends, _half(2.0 ** k))
    _check(torch.tensor([2.0 ** 20], device="cuda"), _half(2.0 ** 20))


@pytest.mark.gpu
def test_fp64_is_within_one_unit_in_the_last_place():
    gen = np.random.default_rng(5)
    g0 = np.concatenate([gen.uniform(-0.5, 1.0, 1 << 19),
                         2.0 ** gen.uniform(-20, 20, 1 << 18) - 1.0]).astype(np.float32)
    g0 = g0[g0 > -1.0]
    src = torch.zeros(g0.size, 9, 1, device="cuda")
    src[:, 0, 0] = torch.as_tensor(g0, device="cuda")
    src[:, 1, 0], src[:, 3, 0] = 1.0, -1.0
    inv = lbm.lbm_channel_profile(src, 0.0).cpu().numpy() / 2.0
    ref = 1.0 / (1.0 + g0.astype(np.float64))
    assert (np.abs(inv - ref) <= np.spacing(ref)).all()
    assert np.mean(inv != ref) < 0.01      # and the quotient itself nearly always


@pytest.mark.gpu
def test_densities_up_to_the_largest_keep_their_momentum():
    """1 / rho is below the smallest normal number from 2^126 on."""
    k = torch.arange(0, 4096, device="cuda", dtype=torch.float64)
    rho = (2.0 ** (120 + 7.999 * k / 4096)).float()
    half = (rho.double() / 16).float()
    src = torch.zeros(1, 9, rho.numel(), device="cuda")
    src[0, 0], src[0, 2], src[0, 4] = rho, half, -half
    g = lbm.lbm_step_bgk(src, torch.empty_like(src), 1.0)[0].double()
    j = (g[2] - g[4]) + (g[5] + g[6] - g[7] - g[8])
    # (FP32 sums of nine terms of the size of rho, and 22 bits of 1 / rho)
    assert float(((j - 2 * half.double()).abs() / rho.double()).max()) <= 1e-5

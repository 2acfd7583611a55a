"""The arithmetic that fp32 attention in bf16 pieces rests on, in numbers of the same formats on the CPU: 2^24 x as three bf16
numbers, and a product of two such without its three smallest partial products."""
import numpy as np
import pytest
import torch


def pieces(x):
    x = x * 2.0 ** 24
    h = x.bfloat16().float()
    m = (x - h).bfloat16().float()
    return x, h, m, (x - h - m).bfloat16().float()


def elements(lo, hi):
    """Numbers of every exponent from lo to hi, the last places of bf16s on either side of them."""
    rng = np.random.default_rng(3)
    x = np.ldexp(1.0 + rng.integers(0, 1 << 23, (hi - lo, 2000)) * 2.0 ** -23, np.arange(lo, hi)[:, None])
    edges = np.ldexp(1.0 + np.array([0, 2.0 ** -8 - 2.0 ** -17, 2.0 ** -8, 2.0 ** -7 - 2.0 ** -23, 2.0 ** -16, 1 - 2.0 ** -23]), np.arange(lo, hi)[:, None])
    return torch.from_numpy(np.concatenate([x, edges], 1).astype(np.float32).ravel())


def test_three_pieces_are_exact():
    """Subnormal numbers (2^-149 and up) and those to 2^103, whose 2^24-fold has finite pieces."""
    x = torch.cat([elements(-126, 103), torch.arange(1, 4096) * 2.0 ** -149, torch.tensor([2.0 ** -126 - 2.0 ** -149])])
    scaled, h, m, l = pieces(torch.cat([x, -x]))
    assert torch.equal(h.double() + m.double() + l.double(), scaled.double())
    # no piece is subnormal
    assert all(((p == 0) | (p.abs() >= 2.0 ** -126)).all() for p in (h, m, l))


@pytest.mark.parametrize("exponents", [(0, 0), (-60, 40), (-126, 30)])
def test_what_six_products_leave_out(exponents):
    """Below 2^-24 of the product; 1 + 2^-8 - 2^-17, rounded up to 1 + 2^-7 where it could lie halfway, comes to 0.99 of that."""
    a, b = (elements(e, e + 1).double() for e in exponents)
    x, y = torch.cartesian_prod(a[-400:], b[-400:]).T
    (_, xh, xm, xl), (_, yh, ym, yl) = (tuple(p.double() for p in pieces(v.float())) for v in (x, y))
    six = xh * yh + xh * ym + xm * yh + xh * yl + xl * yh + xm * ym
    left_out = (xm * yl + xl * ym + xl * yl).abs() / (x * y * 2.0 ** 48)
    assert left_out.max() < 2.0 ** -24
    assert ((six * 2.0 ** -48 - x * y).abs() / (x * y)).max() < 2.0 ** -24
    worst = torch.tensor([1.0 + 2.0 ** -8 - 2.0 ** -17]).float()
    _, h, m, l = (p.double().item() for p in pieces(worst))
    assert 0.9 < abs(2 * m * l + l * l) / (worst.double().item() ** 2 * 2.0 ** 48) / 2.0 ** -24 < 1

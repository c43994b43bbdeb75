"""Scaled harmonics far from the origin: values past the type's range leave the
derivatives that are within it as they are."""
import numpy as np
import pytest
import torch

from _gpu_common import TOL, to_dev

pytestmark = pytest.mark.gpu

# towards the axes, in the planes and across; powers of two scale them exactly
BASE = [[1.0, 0.0, 0.0], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0], [0.0, 0.0, -1.0], [1.0, 1.0, 0.0], [0.6, -0.3, 0.74],
        [-0.25, 0.5, -0.125], [1e-4, 1e-4, 1.0], [1.0, 1.0, 1e-6]]
EXPONENTS = {torch.float32: [10, 17, 33, 50, 63, 66, 83, 126], torch.float64: [30, 60, 260, 510, 515, 700, 1000]}


def _check_degree(got, base, power, e, dt, label):
    """got = base * 2^(e power), for the points whose largest entry of the
    degree is a number of the type (an entry is a sum of terms of that size):
    both carry an error of at most TOL of it."""
    size = np.abs(base).reshape(len(base), -1).max(1)
    with np.errstate(over="ignore"):
        fits = np.ldexp(size, e * power) < float(torch.finfo(dt).max) * 2.0 ** -20
    size = size.reshape(-1, *[1] * (base.ndim - 1))
    got, base, size = got[fits], base[fits], size[fits]
    bad = ~(np.abs(got - np.ldexp(base, e * power)) <= np.ldexp(2 * TOL[dt] * size, e * power))
    assert not bad.any(), (label, np.argwhere(bad)[:5], got[bad][:5], np.ldexp(base, e * power)[bad][:5])


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("l_max", [1, 2, 3, 5, 6, 8, 12, 13, 20])
def test_hessian_entries_within_range(l_max, dt):
    """The Hessian of degree l is homogeneous of degree l - 2."""
    import paper_2302_08381_amd as sph
    x = to_dev(np.asarray(BASE), dt)
    H = sph.sph_compute_with_hessians(x, l_max, False)[2].double().cpu().numpy()
    for e in EXPONENTS[dt]:
        print(f"far Hessians {dt} l_max={l_max} 2^{e}", flush=True)
        F = sph.sph_compute_with_hessians(x * 2.0 ** e, l_max, False)[2].double().cpu().numpy()
        for l in range(l_max + 1):
            k = slice(l * l, (l + 1) ** 2)
            _check_degree(F[..., k], H[..., k], l - 2, e, dt, (l_max, e, l))


@pytest.mark.parametrize("dt,l_max", [(torch.float32, 13), (torch.float32, 16), (torch.float32, 32), (torch.float64, 9),
                                      (torch.float64, 12), (torch.float64, 20)])
def test_double_backward_within_range(dt, l_max):
    """Degrees past the compile-time ones: ggY of degree l is homogeneous of
    degree l - 1, and gxyz2 of a gY in that degree alone of degree l - 2."""
    import paper_2302_08381_amd as sph
    K = (l_max + 1) ** 2
    x = to_dev(np.asarray(BASE), dt)
    rng = np.random.default_rng(2100 + l_max)
    v = to_dev(rng.standard_normal((len(BASE), 3)), dt)
    gY = to_dev(rng.standard_normal((len(BASE), K)), dt)
    gg = sph.sph_double_backward(x, gY, v, l_max, False)[0].double().cpu().numpy()
    for e in EXPONENTS[dt]:
        print(f"far double backward {dt} l_max={l_max} 2^{e}", flush=True)
        fg = sph.sph_double_backward(x * 2.0 ** e, gY, v, l_max, False)[0].double().cpu().numpy()
        for l in range(l_max + 1):
            _check_degree(fg[:, l * l:(l + 1) ** 2], gg[:, l * l:(l + 1) ** 2], l - 1, e, dt, (l_max, e, l))
    # the power at which every degree's second derivatives are within the type's
    # range and the largest degree's harmonics are past it
    emax = torch.finfo(dt).max
    e = int((np.log2(emax) - 16) / (l_max - 2))
    want, size = np.zeros((len(BASE), 3)), np.zeros((len(BASE), 1))
    for l in range(l_max + 1):
        one = torch.zeros_like(gY)
        one[:, l * l:(l + 1) ** 2] = gY[:, l * l:(l + 1) ** 2]
        g2 = sph.sph_double_backward(x, one, v, l_max, False)[1].double().cpu().numpy()
        want += np.ldexp(g2, e * (l - 2))
        size += np.ldexp(np.abs(g2).max(1, keepdims=True), e * (l - 2))
    got = sph.sph_double_backward(x * 2.0 ** e, gY, v, l_max, False)[1].double().cpu().numpy()
    fits = size[:, 0] < emax * 2.0 ** -4
    assert fits.any()
    assert (np.abs(got - want) <= 2 * TOL[dt] * size)[fits].all(), (l_max, e, got, want)


@pytest.mark.parametrize("axis", [0, 2])
@pytest.mark.parametrize("dt,l_max", [(torch.float32, 12), (torch.float32, 13), (torch.float64, 8), (torch.float64, 9)])
def test_double_backward_of_infinite_v(dt, l_max, axis):
    """The columns of order 0, whose factor has no gradient, take an infinite v
    to the infinity of their derivative's sign."""
    import paper_2302_08381_amd as sph
    x = to_dev(np.asarray([[0.3, 0.2, 0.7], [-0.5, 0.1, 0.4]]), dt)
    v = torch.zeros_like(x)
    v[:, axis] = float("inf")
    gY = torch.ones((2, (l_max + 1) ** 2), dtype=dt, device="cuda")
    gg = sph.sph_double_backward(x, gY, v, l_max, False)[0]
    d = sph.sph_compute_with_gradients(x, l_max, False)[1][:, axis]
    for l in range(1 if axis == 2 else 2, l_max + 1):  # (degree 1 has no derivative along x at order 0)
        k = l * l + l
        assert torch.equal(gg[:, k], torch.sign(d[:, k]) * float("inf")), (l, gg[:, k], d[:, k])


@pytest.mark.parametrize("dt,l_max", [(torch.float32, 12), (torch.float32, 13), (torch.float32, 32), (torch.float64, 8),
                                      (torch.float64, 9)])
def test_double_backward_next_to_the_origin(dt, l_max):
    """gxyz2 of the normalised harmonics, homogeneous of degree -2, past the
    type's range: the infinity of its sign."""
    import paper_2302_08381_amd as sph
    rng = np.random.default_rng(2200 + l_max)
    x = to_dev(rng.uniform(0.25, 1.0, (40, 3)) * rng.choice([-1.0, 1.0], (40, 3)), dt)
    v = to_dev(rng.standard_normal((40, 3)), dt)
    gY = to_dev(rng.standard_normal((40, (l_max + 1) ** 2)), dt)
    e = {torch.float32: -70, torch.float64: -530}[dt]
    base = sph.sph_double_backward(x, gY, v, l_max, True)[1]
    got = sph.sph_double_backward(x * 2.0 ** e, gY, v, l_max, True)[1]
    big = base.abs() > 2.0  # times 2^140 or 2^1060; far above the errors of either
    assert int(big.sum()) > 60
    assert torch.equal(got[big], torch.sign(base[big]) * float("inf"))

"""The backward from the points (sph_vector_jacobian) at the edges of its tiles
and on both sides of the compile-time kernels."""
import numpy as np
import pytest
import torch

import oracle
from workloads import standard_normal, standard_normal_points

from _gpu_common import TOL, assert_bitwise_equal, host_points, to_dev

pytestmark = pytest.mark.gpu


def _points(n, seed, normalize):
    pts = standard_normal_points(n, seed)
    special = [[0.0, 0.0, 0.0], [0.0, 0.0, 1.25], [0.0, 0.0, -0.75], [1e-8, -1e-9, 1.0]]
    k = min(n - 1, len(special))
    if k:
        pts[:k] = special[:k]
    return pts if normalize else pts * (0.8 / np.abs(pts).max())  # bounded r^l


def _misaligned(t):
    """The same values one element past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("normalize", [True, False])
@pytest.mark.parametrize("l_max", [0, 1, 3, 4, 7, 8, 9, 12, 13, 16, 31, 32])
def test_vector_jacobian_matches_oracle(l_max, normalize, dtype):
    """One and two waves' tiles, ragged tiles, odd and even K, both sides of
    the compile-time kernels; the same product as the oracle's contraction."""
    import paper_2302_08381_amd as sph
    K = (l_max + 1) ** 2
    for n in (1, 63, 64, 65, 131):
        print(f"vjp l_max={l_max} normalize={normalize} {dtype} n={n}", flush=True)
        xyz = to_dev(_points(n, 7000 + l_max, normalize), dtype)
        gY = to_dev(standard_normal((n, K), 7100 + l_max), dtype)
        gx = sph.sph_vector_jacobian(xyz, gY, l_max, normalize)
        gm = sph.sph_vector_jacobian(_misaligned(xyz), _misaligned(gY), l_max, normalize)
        torch.cuda.synchronize()
        hp, gYh = host_points(xyz), gY.cpu().double().numpy()
        _, Gr = oracle.real_sph(hp, l_max, normalize)
        _, g, _ = oracle.component_scales(hp, l_max, normalize)
        scale = (np.abs(gYh) * g).sum(1)[:, None] + 1e-30
        err = np.abs(gx.cpu().double().numpy() - np.asarray(oracle.backward(Gr, gYh), float)) / scale
        assert np.isfinite(err).all() and err.max() <= TOL[dtype], (n, err.max())
        assert_bitwise_equal(gm, gx, f"misaligned, n={n}")


def test_vector_jacobian_keeps_infinite_gradients():
    """An infinite upstream gradient gives the signed infinity that the
    contraction of stored derivatives gives, a NaN one gives NaN."""
    import paper_2302_08381_amd as sph
    for l_max in (3, 8, 20):
        xyz = to_dev(standard_normal_points(64, 7300), torch.float32)
        gY = to_dev(standard_normal((64, (l_max + 1) ** 2), 7301), torch.float32)
        gY[:20, 2] = float("inf")
        gY[20:40, 1] = float("-inf")
        gY[40:50, 3] = float("nan")
        _, dY = sph.sph_compute_with_gradients(xyz, l_max, True)
        a, b = sph.sph_vector_jacobian(xyz, gY, l_max, True), sph.sph_backward(dY, gY, l_max)
        torch.cuda.synchronize()
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        assert torch.equal(a[torch.isinf(b)], b[torch.isinf(b)])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("normalization", ["integral", "component", "norm"])
@pytest.mark.parametrize("l_max", [0, 2, 8, 12, 13])
def test_e3nn_forms_match_the_conversion(l_max, normalization, dtype):
    """Factors applied while the values and derivatives are formed, against
    the separate conversion of this library's outputs: both round each value
    a few times, well inside the per-degree tolerance."""
    import paper_2302_08381_amd as sph
    n, K = 70, (l_max + 1) ** 2
    xyz = to_dev(_points(n, 7400 + l_max, True), dtype)
    xyz[3] = torch.tensor([0.0, 2.0, 0.0], dtype=dtype)  # e3nn's polar axis
    gY = to_dev(standard_normal((n, K), 7401), dtype)
    Yr, dYr = sph.e3nn_spherical_harmonics_with_gradients(xyz, l_max, True, normalization)
    gr = sph.sph_backward(dYr, gY, l_max)
    x = xyz.clone().requires_grad_(True)
    Y = sph.e3nn_spherical_harmonics(x, l_max, True, normalization)
    with torch.no_grad():
        x.mul_(3.0)  # the backward's points are the forward's, whatever becomes of the caller's tensor
    (g,) = torch.autograd.grad(Y, x, gY)
    torch.cuda.synchronize()
    hp, gYh = host_points(xyz[:, [2, 0, 1]].contiguous()), gY.abs().cpu().double().numpy()
    s, gs, _ = oracle.component_scales(hp, l_max, True)
    c = np.sqrt(4 * np.pi)  # the largest factor
    assert (np.abs((Y.detach() - Yr).cpu().double().numpy()) / (c * s)).max() <= TOL[dtype]
    scale = c * (gYh * gs).sum(1)[:, None] + 1e-30
    assert (np.abs((g - gr).cpu().double().numpy()) / scale).max() <= TOL[dtype]

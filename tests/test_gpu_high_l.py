"""The kernels of the degrees past the compile-time ones, at the edges of their
tiles."""
import numpy as np
import pytest
import torch

import oracle
from workloads import standard_normal_points

from _gpu_common import TOL, assert_close_per_l, host_points, to_dev

pytestmark = pytest.mark.gpu


def _points(n, seed, normalize):
    pts = standard_normal_points(n, seed)
    special = [[0.0, 0.0, 0.0], [0.0, 0.0, 1.25], [0.0, 0.0, -0.75], [1e-8, -1e-9, 1.0]]
    k = min(n - 1, len(special))
    if k:
        pts[:k] = special[:k]
    return pts if normalize else pts * (0.8 / np.abs(pts).max())  # bounded r^l


@pytest.mark.parametrize("dtype,l_max", [(torch.float32, 13), (torch.float32, 15), (torch.float32, 32),
                                         (torch.float64, 9), (torch.float64, 16), (torch.float64, 31)])
@pytest.mark.parametrize("normalize", [True, False])
def test_high_degree_tiles(dtype, l_max, normalize):
    """Every count of points of the last tile, values and derivatives, with
    outputs at every offset from a 16-byte boundary."""
    import paper_2302_08381_amd as sph
    K = (l_max + 1) ** 2
    W = 16 // torch.empty((), dtype=dtype).element_size()
    pts = _points(40, 7200 + l_max, normalize)
    hp = host_points(to_dev(pts, dtype))
    Yr, Gr = oracle.real_sph(hp, l_max, normalize)
    for n in list(range(1, 18)) + [40]:
        xyz = to_dev(pts[:n], dtype)
        shift = n % W
        ybuf = torch.full((n * K + 2 * W,), 7.0, dtype=dtype, device="cuda")
        dbuf = torch.full((3 * n * K + 2 * W,), 7.0, dtype=dtype, device="cuda")
        Y, dY = ybuf[shift:shift + n * K].view(n, K), dbuf[shift:shift + 3 * n * K].view(n, 3, K)
        sph.sph_compute_with_gradients(xyz, l_max, normalize, Y=Y, dY=dY)
        V = sph.sph_compute(xyz, l_max, normalize)
        torch.cuda.synchronize()
        assert_close_per_l(Y.cpu().numpy(), Yr[:n], hp[:n], l_max, normalize, "Y", TOL[dtype], f"n={n}")
        assert_close_per_l(dY.cpu().numpy(), Gr[:n], hp[:n], l_max, normalize, "dY", TOL[dtype], f"n={n}")
        assert_close_per_l(V.cpu().numpy(), Yr[:n], hp[:n], l_max, normalize, "Y", TOL[dtype], f"values, n={n}")
        # nothing written outside the outputs
        assert bool((ybuf[:shift] == 7).all()) and bool((ybuf[shift + n * K:] == 7).all())
        assert bool((dbuf[:shift] == 7).all()) and bool((dbuf[shift + 3 * n * K:] == 7).all())

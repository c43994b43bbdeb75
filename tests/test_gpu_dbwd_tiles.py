"""Double backward at the edges of its kernels: ragged last tiles, one, two and
four waves per tile, the last compile-time and the first run-time degrees,
tiles padded in LDS (odd l_max), arrays off 16-byte boundaries, nothing written
outside the outputs, and infinite upstream gradients."""
import numpy as np
import pytest
import torch

import oracle
from workloads import shell_points, standard_normal

from _gpu_common import TOL, assert_bitwise_equal, host_points, to_dev
from test_gpu_backward import _rel_err_vec

pytestmark = pytest.mark.gpu


def _shifted(t, shift):
    """A copy of t that starts `shift` elements past a 256-byte boundary."""
    buf = torch.full((t.numel() + 64,), -7.0, dtype=t.dtype, device=t.device)
    out = buf[16 + shift:16 + shift + t.numel()].view(t.shape)
    out.copy_(t)
    return buf, out


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 63, 130])
@pytest.mark.parametrize("l_max", [0, 1, 2, 5, 7, 8, 9, 10, 11, 12, 13, 16, 17])
def test_double_backward_tiles(l_max, n, dtype):
    import paper_2302_08381_amd as sph
    normalize = (l_max + n) % 2 == 0
    print(f"double backward tiles l_max={l_max} n={n} {dtype} normalize={normalize}", flush=True)
    K = (l_max + 1) ** 2
    xyz = to_dev(shell_points(n, 0.5, 5.0 if normalize else 1.6, 1400 + l_max), dtype)
    gY = to_dev(standard_normal((n, K), 1500 + l_max), dtype)
    v = to_dev(standard_normal((n, 3), 1600 + l_max), dtype)
    ggY, g2 = sph.sph_double_backward(xyz, gY, v, l_max, normalize)
    for a, b in ((1, 1), (0, 1), (2, 3)):
        _, gs = _shifted(gY, a)
        buf, out = _shifted(gY, b)
        gg, h = sph.sph_double_backward(xyz, gs, v, l_max, normalize, grad_grad_Y=out)
        torch.cuda.synchronize()
        assert bool((buf[:16 + b] == -7.0).all()) and bool((buf[16 + b + n * K:] == -7.0).all())
        assert_bitwise_equal(gg, ggY, f"ggY at offsets {a}, {b}")
        assert_bitwise_equal(h, g2, f"gxyz2 at offsets {a}, {b}")
    hp = host_points(xyz)
    gYh, vh = gY.cpu().double().numpy(), v.cpu().double().numpy()
    ggr, g2r = oracle.double_backward(hp, gYh, vh, l_max, normalize)
    _, g, h = oracle.component_scales(hp, l_max, normalize)
    vn = np.sqrt((vh ** 2).sum(1))[:, None]
    assert _rel_err_vec(ggY.cpu().numpy(), ggr, g * vn).max() <= TOL[dtype]
    s2 = (np.abs(gYh) * h).sum(1)[:, None] * vn
    assert _rel_err_vec(g2.cpu().numpy(), g2r, s2).max() <= TOL[dtype]
    # each output alone
    a, b = sph.sph_double_backward(xyz, gY, v, l_max, normalize, want_grad_xyz=False)
    assert b is None and torch.equal(a, ggY)
    a, b = sph.sph_double_backward(xyz, gY, v, l_max, normalize, want_grad_grad_Y=False)
    assert a is None and torch.equal(b, g2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("normalize", [False, True])
def test_double_backward_infinite_gradient(normalize, dtype):
    """An infinite entry of gY gives its product with H_k v at its own point,
    by sign, and leaves every other value as it was."""
    import paper_2302_08381_amd as sph
    l_max, n, i, k = 14, 40, 7, 101
    xyz = to_dev(shell_points(n, 0.5, 1.5, 1700), dtype)
    gY = to_dev(standard_normal((n, (l_max + 1) ** 2), 1701), dtype)
    v = to_dev(standard_normal((n, 3), 1702), dtype)
    gg0, h0 = sph.sph_double_backward(xyz, gY, v, l_max, normalize)
    _, _, H = sph.sph_compute_with_hessians(xyz, l_max, normalize)
    gY[i, k] = float("inf")
    gg, h = sph.sph_double_backward(xyz, gY, v, l_max, normalize)
    torch.cuda.synchronize()
    assert torch.equal(gg, gg0)
    keep = torch.arange(n, device="cuda") != i
    assert torch.equal(h[keep], h0[keep])
    want = H[i, :, :, k].double() @ v[i].double()
    assert bool(torch.isinf(h[i]).all()) and torch.equal(torch.sign(h[i]).double(), torch.sign(want))

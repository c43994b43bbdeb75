"""Explicit second derivatives at the edges of the Hessian kernel's tiles:
ragged last tiles, one and two lanes per (point, order), compile-time and
run-time degrees, rows padded in LDS (odd l_max), outputs off a 16-byte
boundary, and nothing written outside the output."""
import numpy as np
import pytest
import torch

import oracle
from workloads import shell_points

from _gpu_common import TOL, assert_bitwise_equal, host_points, to_dev
from test_gpu_hessian import _hess_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 63, 66])
@pytest.mark.parametrize("l_max", [0, 1, 5, 6, 7, 8, 9, 11, 12, 13, 16, 17])
def test_hessian_tiles(l_max, n, dtype):
    import paper_2302_08381_amd as sph
    normalize = (l_max + n) % 2 == 0
    print(f"hessian tiles l_max={l_max} n={n} {dtype} normalize={normalize}", flush=True)
    xyz = to_dev(shell_points(n, 0.5, 5.0 if normalize else 1.6, 1300 + l_max), dtype)
    K = (l_max + 1) ** 2
    cnt = n * 9 * K
    outs = []
    for shift in range(4):
        buf = torch.full((cnt + 64,), -7.0, dtype=dtype, device="cuda")
        d2Y = buf[16 + shift:16 + shift + cnt].view(n, 3, 3, K)
        sph.sph_compute_with_hessians(xyz, l_max, normalize, store_dY=False, d2Y=d2Y)
        torch.cuda.synchronize()
        assert bool((buf[:16 + shift] == -7.0).all()) and bool((buf[16 + shift + cnt:] == -7.0).all())
        outs.append(d2Y)
    for shift in range(1, 4):
        assert_bitwise_equal(outs[shift], outs[0], f"offset {shift}")
    hp = host_points(xyz)
    _, _, H = oracle.definition_eval_ld(hp, l_max, normalize, hessian=True)
    got = outs[0].cpu().numpy()
    err = _hess_err(got, H, hp, l_max, normalize)
    assert np.isfinite(got).all() and err <= TOL[dtype], err
    assert np.array_equal(got, got.transpose(0, 2, 1, 3))

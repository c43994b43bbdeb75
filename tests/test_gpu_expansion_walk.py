"""The compile-time backward of the radial expansion at the edges of its walk:
chunks of up to 64 points through up to four environments, windows of 64
environments."""
import numpy as np
import pytest
import torch

from workloads import standard_normal

from _gpu_common import host_points, to_dev
from test_gpu_expansion import _case, _check_backward

pytestmark = pytest.mark.gpu

COUNTS = {
    # chunks that take one to four environments and stop at the fourth's end,
    # at 64 points exactly, and one point to either side
    "slices": [1, 1, 1, 1, 1, 2, 3, 4, 16, 16, 16, 16, 63, 1, 64, 62, 1, 1, 65, 20, 20, 20, 20, 20],
    # empty environments past one window, at both ends and inside
    "empties": [0] * 70 + [5] + [0] * 200 + [3, 0, 0, 130] + [0] * 63 + [2] + [0] * 64 + [1] + [0] * 90,
    "one": [1],
    "long": [700],
}


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("l_max,n_max", [(0, 8), (3, 8), (4, 5), (5, 16), (8, 8), (7, 16), (12, 8), (9, 12)])
@pytest.mark.parametrize("counts", sorted(COUNTS))
def test_backward_walk(counts, l_max, n_max, dt):
    import paper_2302_08381_amd as sph
    print(f"expansion backward walk {counts} l_max={l_max} n_max={n_max} {dt}", flush=True)
    pts, offs, R = _case(COUNTS[counts], l_max, n_max, 1700 + l_max)
    xyz, Rt = to_dev(pts, dt), to_dev(R, dt)
    Gt = to_dev(standard_normal((offs.size - 1, n_max, (l_max + 1) ** 2), 1701), dt)
    o = torch.as_tensor(offs, device="cuda")
    gx, gR = sph.sph_radial_expansion_backward(xyz, o, Rt, Gt, l_max, True)
    only_R = sph.sph_radial_expansion_backward(xyz, o, Rt, Gt, l_max, True, want_grad_xyz=False)[1]
    torch.cuda.synchronize()
    assert torch.equal(only_R, gR)
    _check_backward(gx, gR, host_points(xyz), offs, Rt.cpu().double().numpy(), Gt.cpu().double().numpy(), l_max, True,
                    dt, f"{counts} {dt} L={l_max} n={n_max}")


def test_backward_inconsistent_offsets_stay_inside():
    """Offsets that decrease, start late or end past the points: reported, and
    nothing outside the arrays is written."""
    import paper_2302_08381_amd as sph
    L, NM, n = 4, 8, 40
    pts, _, R = _case([n], L, NM, 1750)
    xyz, Rt = to_dev(pts, torch.float32), to_dev(R, torch.float32)
    for bad in ([0, 25, 10, n], [3, 9, 30, n], [0, 10, 20, 500], [0, -5, 70, 12]):
        G = to_dev(standard_normal((3, NM, (L + 1) ** 2), 1751), torch.float32)
        st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        sph.sph_radial_expansion_backward(xyz, torch.tensor(bad, device="cuda"), Rt, G, L, True, status=st)
        torch.cuda.synchronize()
        assert int(st.item()) == 4

"""The compile-time radial expansion and its backward at the edges of their
walks: chunks of up to 64 (or 32) points, in the backward through up to four
environments, windows of 64 environments."""
import numpy as np
import pytest
import torch

from workloads import standard_normal

from _gpu_common import host_points, to_dev
from test_gpu_expansion import _case, _check, _check_backward

pytestmark = pytest.mark.gpu

COUNTS = {
    # chunks that take one to four environments and stop at the fourth's end,
    # at 64 points exactly, and one point to either side
    "slices": [1, 1, 1, 1, 1, 2, 3, 4, 16, 16, 16, 16, 63, 1, 64, 62, 1, 1, 65, 20, 20, 20, 20, 20],
    # empty environments past one window, at both ends and inside
    "empties": [0] * 70 + [5] + [0] * 200 + [3, 0, 0, 130] + [0] * 63 + [2] + [0] * 64 + [1] + [0] * 90,
    "one": [1],
    "long": [700],
    # enough environments for the two-wave blocks of low degrees
    "many": [3, 1, 0, 2, 70] * 120,
}


# both sides of the channel layouts (4, 8, 12, 16 channels), of the degrees at
# which three groups of four need more than the block's threads, and of the
# largest degrees and channels that the compile-time kernel takes
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("l_max,n_max", [(0, 1), (0, 16), (1, 4), (3, 9), (5, 8), (6, 5), (4, 6), (7, 6), (8, 6), (8, 9), (8, 12), (8, 16), (9, 3), (11, 12),
                                         (12, 12), (12, 16), (13, 8), (4, 17)])
@pytest.mark.parametrize("counts", sorted(COUNTS))
def test_forward_walk(counts, l_max, n_max, dt):
    import paper_2302_08381_amd as sph
    print(f"expansion walk {counts} l_max={l_max} n_max={n_max} {dt}", flush=True)
    pts, offs, R = _case(COUNTS[counts], l_max, n_max, 1800 + l_max)
    xyz, Rt, o = to_dev(pts, dt), to_dev(R, dt), torch.as_tensor(offs, device="cuda")
    c = torch.full((offs.size - 1, n_max, (l_max + 1) ** 2), float("nan"), dtype=dt, device="cuda")
    sph.sph_radial_expansion(xyz, o, Rt, l_max, l_max % 2 == 0, out=c)
    again = sph.sph_radial_expansion(xyz, o, Rt, l_max, l_max % 2 == 0)
    torch.cuda.synchronize()
    assert torch.equal(c, again)
    _check(c, host_points(xyz), offs, Rt.cpu().double().numpy(), l_max, l_max % 2 == 0, dt,
           f"{counts} {dt} L={l_max} n={n_max}")


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("l_max,n_max", [(0, 8), (3, 8), (4, 5), (5, 16), (8, 8), (7, 16), (10, 5), (11, 8), (12, 8), (9, 12)])
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
        sph.sph_radial_expansion(xyz, torch.tensor(bad, device="cuda"), Rt, L, True, status=st.fill_(-1))
        torch.cuda.synchronize()
        assert int(st.item()) == 4

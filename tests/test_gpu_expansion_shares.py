"""How the radial expansion's blocks share the environments: a run of empty
ones is spread over them."""
import numpy as np
import pytest
import torch

from workloads import standard_normal

from _gpu_common import host_points, to_dev
from test_gpu_expansion import _case, _check, _check_backward

pytestmark = pytest.mark.gpu


def _us(f, reps=5):
    f()
    best = float("inf")
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3)
    return best


# the low degrees, the padded channels and the run-time degrees
@pytest.mark.parametrize("l_max,n_max", [(3, 8), (8, 5), (14, 8)])
@pytest.mark.parametrize("where", ["all", "tail", "middle", "head"])
def test_empty_environments_are_spread(where, l_max, n_max):
    """30 000 environments, nearly all empty: no more time than three times
    what 30 000 environments of one point take (all of the empty ones in one
    block take 20 times as long as those or more)."""
    import paper_2302_08381_amd as sph
    n_env = 30000
    counts = np.zeros(n_env, np.int64)
    if where != "all":
        at = {"tail": 0, "middle": n_env // 2, "head": n_env - 40}[where]
        counts[at:at + 40] = np.arange(1, 41)
    pts, offs, R = _case(counts, l_max, n_max, 1900 + l_max)
    xyz, Rt, o = to_dev(pts, torch.float32), to_dev(R, torch.float32), torch.as_tensor(offs, device="cuda")
    one = torch.arange(n_env + 1, device="cuda")
    x1 = torch.randn((n_env, 3), device="cuda")
    R1 = torch.randn((n_env, l_max + 1, n_max), device="cuda")
    print(f"expansion shares {where} l_max={l_max} n_max={n_max}", flush=True)
    c = torch.full((n_env, n_max, (l_max + 1) ** 2), float("nan"), device="cuda")
    t = _us(lambda: sph.sph_radial_expansion(xyz, o, Rt, l_max, out=c, check=False))
    t1 = _us(lambda: sph.sph_radial_expansion(x1, one, R1, l_max, out=torch.empty_like(c), check=False))
    assert t < 3 * t1, (t, t1)
    full = counts > 0
    assert not bool(c[torch.as_tensor(~full, device="cuda")].any())
    if where != "all":
        kept = np.concatenate([[0], np.cumsum(counts[full])])
        _check(c[torch.as_tensor(full, device="cuda")], host_points(xyz), kept, Rt.cpu().double().numpy(), l_max, True,
               torch.float32, where)


# both sides of the counts of environments at which the waves change (512 is
# two a CU), and of eight
@pytest.mark.parametrize("n_env", [1, 2, 7, 8, 9, 17, 511, 512, 513, 600])
@pytest.mark.parametrize("dt,l_max,n_max", [(torch.float32, 3, 8), (torch.float32, 4, 5), (torch.float64, 3, 16),
                                            (torch.float64, 1, 12), (torch.float64, 4, 5), (torch.float64, 4, 8),
                                            (torch.float64, 5, 8), (torch.float64, 5, 7)])
def test_shares_of_few_environments(dt, l_max, n_max, n_env):
    import paper_2302_08381_amd as sph
    print(f"expansion shares {n_env} {dt} l_max={l_max} n_max={n_max}", flush=True)
    counts = np.arange(n_env) * 7 % 5  # 0 .. 4 points
    counts[0] = 70
    pts, offs, R = _case(counts, l_max, n_max, 1950 + n_env)
    xyz, Rt, o = to_dev(pts, dt), to_dev(R, dt), torch.as_tensor(offs, device="cuda")
    c = torch.full((n_env, n_max, (l_max + 1) ** 2), float("nan"), dtype=dt, device="cuda")
    sph.sph_radial_expansion(xyz, o, Rt, l_max, out=c)
    hp, hR = host_points(xyz), Rt.cpu().double().numpy()
    _check(c, hp, offs, hR, l_max, True, dt, f"{n_env}")
    G = to_dev(standard_normal(tuple(c.shape), 1951), dt)
    gx, gR = sph.sph_radial_expansion_backward(xyz, o, Rt, G, l_max, True)
    _check_backward(gx, gR, hp, offs, hR, G.cpu().double().numpy(), l_max, True, dt, f"{n_env}")


@pytest.mark.parametrize("per", [127, 128])
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
def test_long_environments_past_two_a_cu(dt, per):
    """The length from which four waves take environments that are resident at
    once, and the one below it."""
    import paper_2302_08381_amd as sph
    n_env, l_max, n_max = 520, 3, 8
    pts, offs, R = _case([per] * n_env, l_max, n_max, 1960)
    xyz, Rt = to_dev(pts, dt), to_dev(R, dt)
    c = sph.sph_radial_expansion(xyz, torch.as_tensor(offs, device="cuda"), Rt, l_max)
    hp, hR = host_points(xyz), Rt.cpu().double().numpy()
    for e in (0, 259, 512, 519):  # the grid's environments one by one
        b = slice(offs[e], offs[e + 1])
        _check(c[e:e + 1], hp[b], np.array([0, per]), hR[b], l_max, True, dt, f"environment {e}")

"""How the radial expansion's blocks share the environments: a run of empty
ones is spread over them."""
import numpy as np
import pytest
import torch

from _gpu_common import host_points, to_dev
from test_gpu_expansion import _case, _check

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

"""The batched path past the compile-time degrees: every variant that can be
pinned, and the bits of a tuned call."""
import numpy as np
import pytest
import torch

import oracle
from workloads import csr_environments, standard_normal

from _gpu_common import TOL, assert_bitwise_equal, assert_close_per_l, host_points, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,l_max", [(torch.float32, 13), (torch.float32, 20), (torch.float32, 32), (torch.float64, 9),
                                      (torch.float64, 16)])
def test_every_variant_matches_oracle(dt, l_max):
    import paper_2302_08381_amd as sph
    pts, offs = csr_environments(12, 8, 64, 0.5, 5.0, 2300 + l_max)
    n, K = int(offs[-1]), (l_max + 1) ** 2
    xyz, o = to_dev(pts, dt), torch.as_tensor(offs, device="cuda")
    gY = to_dev(standard_normal((n, K), 2301 + l_max), dt)
    hp = host_points(xyz)
    Yr, Gr = oracle.real_sph(hp, l_max, True)
    gref = np.asarray(oracle.backward(Gr, gY.cpu().double().numpy()), float)
    _, gsc, _ = oracle.component_scales(hp, l_max, True)
    gscale = (gY.abs().cpu().double().numpy() * gsc).sum(1)[:, None]
    for store_dY, bwd in ((True, True), (True, False), (False, True)):
        ran = []
        for variant in ("default", "runtime_degree", "degree_split"):
            print(f"batched variant {dt} l_max={l_max} {variant} dY={store_dY} backward={bwd}", flush=True)
            try:
                sph.sph_batched_set_config(l_max, True, dt, store_dY, bwd, variant, 0)
            except sph.SphError:
                continue
            ran.append(variant)
            out = sph.sph_batched_compute(xyz, o, l_max, True, store_dY=store_dY, grad_Y=gY if bwd else None)
            assert_close_per_l(out["Y"].cpu().numpy(), Yr, hp, l_max, True, "Y", TOL[dt], variant)
            if store_dY:
                assert_close_per_l(out["dY"].cpu().numpy(), Gr, hp, l_max, True, "dY", TOL[dt], variant)
            if bwd:
                err = np.abs(out["grad_xyz"].cpu().double().numpy() - gref) / gscale
                assert err.max() <= TOL[dt], (variant, err.max())
        sph.sph_batched_set_config(l_max, True, dt, store_dY, bwd, "default", 0)
        assert ran == ["default", "runtime_degree"] + ([] if bwd else ["degree_split"])


@pytest.mark.parametrize("dt,l_max", [(torch.float32, 14), (torch.float64, 10)])
def test_tuned_call_has_the_plain_call_s_bits(dt, l_max):
    import paper_2302_08381_amd as sph
    n = 64 * 256 + 5
    xyz = torch.randn((n, 3), device="cuda", dtype=dt)
    gY = torch.randn((n, (l_max + 1) ** 2), device="cuda", dtype=dt)
    o = torch.tensor([0, n], device="cuda")
    Y, dY = sph.sph_compute_with_gradients(xyz, l_max, False)
    for store_dY in (False, True):
        for bwd in (False, True):
            out = sph.sph_batched_compute(xyz, o, l_max, False, store_dY=store_dY, grad_Y=gY if bwd else None)
            assert "kernel=default " in sph.sph_batched_get_config(l_max, False, dt, store_dY, bwd)
            assert_bitwise_equal(out["Y"], Y, f"Y {store_dY} {bwd}")
            if store_dY:
                assert_bitwise_equal(out["dY"], dY, f"dY {bwd}")

"""Frames cut into even tiles at the edges of the default and explicit tile
sizes: the reduced system against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ba64
from scenes import tiny_scene

pytestmark = pytest.mark.gpu


# one patch; one full tile, two even ones and three around each precision's
# default (56 in float64, 96 in float32); explicit sizes, the last not a divisor
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("patches,cap", [(1, 0), (56, 0), (57, 0), (96, 0), (97, 0), (113, 0), (33, 32), (50, 7)])
def test_reduced_system_of_even_tiles(prec, patches, cap):
    import paper_2408_01654_amd as dp

    s = tiny_scene(6, patches, seed=3, radius=3)
    pb = ba64.Problem.from_scene(s)
    ne = ba64.normal_equations(pb, ba64.edge_terms(pb, z_min=s.z_min))
    rs = ba64.reduce(ne, s.lam)
    dt = torch.float64 if prec == "fp64" else torch.float32
    ctx = dp.Context(0)
    try:
        g = dp.GraphTensors.from_scene(s)
        ctx.analyze(g, tile_patches_fp32=cap, tile_patches_fp64=cap)
        poses = torch.as_tensor(s.poses, dtype=dt).cuda()
        depth = torch.as_tensor(s.inv_depth, dtype=dt).cuda()
        print(f"even tiles {prec} {patches} {cap}", flush=True)
        S, sv, _ = ctx.reduced_system(g, poses, depth, lam=s.lam, z_min=s.z_min,
                                      precision=dp.FP64 if prec == "fp64" else dp.FP32)
        # rounding of sums with cancellation (terms up to ~1e3 x |S|)
        tol = 1e-11 if prec == "fp64" else 2e-5
        assert np.abs(S.double().cpu().numpy() - rs.S).max() < tol * np.abs(rs.S).max()
        assert np.abs(sv.double().cpu().numpy() - rs.s).max() < tol * np.abs(rs.s).max()
    finally:
        ctx.close()

"""A graph whose one-patch tiles carry their padding beyond the shared-memory
budget (every patch seen in 44 other frames): analysed, and its reduced
system and solve against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ba64
from scenes import tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fixed", [0, 1])  # 44 slots with 45 and with 44 free blocks
def test_one_patch_tiles_at_the_limit(n_fixed):
    import paper_2408_01654_amd as dp

    s = tiny_scene(45, 2, seed=5, radius=45, n_fixed=n_fixed, trajectory="forward")
    pb = ba64.Problem.from_scene(s)
    ne = ba64.normal_equations(pb, ba64.edge_terms(pb, z_min=s.z_min))
    rs = ba64.reduce(ne, s.lam)
    want = ba64.solve_scene(s)[2].cost
    ctx = dp.Context(0)
    try:
        g = dp.GraphTensors.from_scene(s)
        print(f"one-patch tiles, {n_fixed} held: analyze", flush=True)
        ctx.analyze(g)
        assert ctx.analysis_info(dp.FP32)["n_tiles"] == 90 and ctx.analysis_info(dp.FP32)["lds_bytes"] > 80 * 1024
        for P, dt, tol in ((dp.FP32, torch.float32, 2e-5), (dp.FP64, torch.float64, 1e-11)):
            poses = torch.as_tensor(s.poses, dtype=dt).cuda()
            depth = torch.as_tensor(s.inv_depth, dtype=dt).cuda()
            print(f"  precision {P}", flush=True)
            S, sv, _ = ctx.reduced_system(g, poses, depth, lam=s.lam, z_min=s.z_min, precision=P)
            # rounding of sums with cancellation (terms up to ~1e3 x |S|)
            assert np.abs(S.double().cpu().numpy() - rs.S).max() < tol * np.abs(rs.S).max()
            assert np.abs(sv.double().cpu().numpy() - rs.s).max() < tol * np.abs(rs.s).max()
            # the cost does not see the free gauge, which the damping alone holds: a step's
            # error enters it through what the edges fix (float32 sums of |r|^2: 1e-7 x 1e3 edges)
            rep = ctx.solve(g, poses, depth, n_iters=2, lam=s.lam, z_min=s.z_min, precision=P)
            assert rep["status"] == 0
            assert np.allclose(rep["cost"], want, rtol=1e-2 if P == dp.FP32 else 1e-6)
    finally:
        ctx.close()

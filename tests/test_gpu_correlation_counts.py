"""3 x 3 patch correlation on both sides of the edge counts where its launch
changes (a few edges of 256 channels by points, a workgroup an edge, four edges
a workgroup), compact and scattered patches mixed, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import correlation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 256])
@pytest.mark.parametrize("E", [1, 96, 97, 512, 513])
def test_edge_counts(D, E):
    import paper_2408_01654_amd as dp

    rng = np.random.default_rng(E + D)
    M, H, W, P = 2, 19, 26, 5
    g = rng.standard_normal((P, 3, 3, D)).astype(np.float32)
    f = rng.standard_normal((M, H, W, D)).astype(np.float32)
    kk, jj = rng.integers(0, P, E), rng.integers(0, M, E)
    centre = np.stack([rng.uniform(-6, W + 6, E), rng.uniform(-6, H + 6, E)], -1)
    grid = np.arange(3) - 1.0
    off = np.stack(np.broadcast_arrays(grid[None, :], grid[:, None]), -1)
    spacing = rng.choice([0.8, 3.0, 6.0, 14.0], E)  # the last two: windows one by one, some of them outside
    xy = (centre[:, None, None, :] + off * spacing[:, None, None, None]).astype(np.float32)
    i32 = lambda a: torch.as_tensor(a.astype(np.int32)).cuda()
    bad = kk.copy()
    bad[E // 2] = P  # zeros for this edge alone, reported
    ctx = dp.Context(0)
    try:
        for idx in (kk, bad):
            print(f"correlation of {E} edges D={D}", flush=True)
            C = ctx.patch_correlation(torch.as_tensor(g).cuda(), torch.as_tensor(f).cuda(), i32(idx), i32(jj),
                                      torch.as_tensor(xy).cuda()).cpu().numpy()
            want = correlation.correlation(g, f, kk, jj, xy)
            # the bound of a float32 dot product of D terms and its interpolation
            bound = (D + 8) * 2.0 ** -24 * correlation.correlation(np.abs(g), np.abs(f), kk, jj, xy) + 1e-30
            ok = np.abs(C - want) <= bound
            if idx is bad:
                assert (C[E // 2] == 0).all()
                ok[E // 2] = True
            assert ok.all()
        assert ctx.device_status() == (dp.binding.DPVBA_EDEVICE, 4)
    finally:
        ctx.close()

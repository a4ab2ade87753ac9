"""Edges of the patch kernels' tiles: the union window of the 3 x 3 patch
correlation (sizes around a 16-pixel tile and around its limit, clipped at
the map's borders, unaligned maps) and the 256-edge groups of the full-patch
reprojection, against the float64 oracles."""
import numpy as np
import pytest
import torch

from oracle import ba64, correlation
from scenes import tiny_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2408_01654_amd as dp
    return dp


@pytest.fixture(scope="module")
def ctx(dp):
    c = dp.Context(0)
    yield c
    c.close()


# spacing of the patch's pixels -> union of 8 + 2 s map pixels a side (limit:
# 256 pixels); the offsets put windows inside, across and outside the borders
@pytest.mark.parametrize("spacing", [0.0, 0.4, 1.0, 3.9, 4.0, 4.2, 9.0])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("shift", [0, 1])
def test_correlation_union_windows(dp, ctx, spacing, D, shift):
    rng = np.random.default_rng(int(10 * spacing) + D)
    E, M, H, W, P = 45, 2, 23, 31, 5
    print(f"correlation spacing {spacing} D={D} shift {shift}", flush=True)
    g = rng.standard_normal((P, 3, 3, D)).astype(np.float32)
    f = rng.standard_normal((M, H, W, D)).astype(np.float32)
    kk, jj = rng.integers(0, P, E), rng.integers(0, M, E)
    centre = np.stack([rng.uniform(-9, W + 9, E), rng.uniform(-9, H + 9, E)], -1)
    centre[0] = (11.0, 9.0)
    centre[1] = (-200.0, 5.0)
    grid = np.arange(3) - 1.0
    off = np.stack(np.broadcast_arrays(grid[None, :], grid[:, None]), -1) * spacing
    xy = (centre[:, None, None, :] + off).astype(np.float32)
    fm = torch.empty(M * H * W * D + 1, device="cuda")[shift:shift + M * H * W * D].reshape(M, H, W, D)
    fm.copy_(torch.as_tensor(f))  # shift 1: rows not aligned to 16 bytes
    i32 = lambda a: torch.as_tensor(a.astype(np.int32)).cuda()
    C = ctx.patch_correlation(torch.as_tensor(g).cuda(), fm, i32(kk), i32(jj), torch.as_tensor(xy).cuda())
    want = correlation.correlation(g, f, kk, jj, xy)
    bound = (D + 8) * 2.0 ** -24 * correlation.correlation(np.abs(g), np.abs(f), kk, jj, xy) + 1e-30
    assert np.all(np.abs(C.cpu().numpy() - want) <= bound)


def test_correlation_non_finite(dp, ctx):
    """A point that is not a number gives no number and one at infinity or
    beyond 1e9 reads no pixel; an infinite feature stays at its own pixel."""
    g = torch.ones(1, 3, 3, 64, device="cuda")
    f = torch.ones(1, 16, 16, 64, device="cuda")
    f[0, 2, 3, 5] = float("inf")
    xy = torch.full((3, 3, 3, 2), 7.0, device="cuda")
    xy[0, 1, 1, 0] = float("nan")
    xy[1, 0, 2] = 3e9
    idx = torch.zeros(3, dtype=torch.int32, device="cuda")
    C = ctx.patch_correlation(g, f, idx, idx, xy).cpu()
    assert torch.isnan(C[0, 1, 1]).all() and torch.isfinite(C[0, 0, 0]).any()
    assert (C[1, 0, 2] == 0).all()
    # (x, y) = (7, 7): sample (a, b) reads pixel (4 + a, 4 + b) with weight one and its neighbours with zero
    assert (C[2] == 64.0).all()


@pytest.mark.parametrize("p", [1, 3, 5])
@pytest.mark.parametrize("n_edges", [1, 255, 256, 257, 700])
def test_reproject_groups_of_edges(dp, ctx, p, n_edges):
    s = tiny_scene(8, 16, seed=5)
    c = s.patches[:, 1:2, 1:2, :].astype(np.float64)
    grid = np.arange(p) - (p - 1) / 2
    off = np.stack(np.broadcast_arrays(grid[None, :], grid[:, None]), -1)
    patches = (c + off).astype(np.float32)
    rng = np.random.default_rng(n_edges)
    e = rng.integers(0, s.n_edges, n_edges)
    g = dp.GraphTensors.from_arrays(s.n_frames, 2, patches, s.ii[e], s.jj[e], s.kk[e], s.target[e], s.weight[e],
                                    s.intrinsics)
    depth = s.inv_depth.copy()
    depth[::7] *= -1.0  # not visible
    print(f"reproject p={p} E={n_edges}", flush=True)
    coords, valid = ctx.reproject(g, torch.as_tensor(s.poses).cuda(), torch.as_tensor(depth).cuda(), z_min=0.1)
    fx, fy, cx, cy = (float(x) for x in s.intrinsics)
    R, t = ba64.relative_poses(s.poses.astype(np.float64), s.ii[e], s.jj[e])
    d = depth.astype(np.float64)[s.kk[e]]
    uv = patches.astype(np.float64)[s.kk[e]]
    ray = np.stack([(uv[..., 0] - cx) / fx, (uv[..., 1] - cy) / fy, np.ones(uv.shape[:-1])], -1)
    q = np.einsum("eab,exyb->exya", R, ray) + (t * d[:, None])[:, None, None, :]
    mag = np.einsum("eab,exyb->exya", np.abs(R), np.abs(ray)) + (np.abs(t) * np.abs(d)[:, None])[:, None, None, :]
    # every factor carries a few float32 roundings: 32 of them on the terms' magnitudes
    for m, (f_, c_) in enumerate(((fx, cx), (fy, cy))):
        want = f_ * q[..., m] / q[..., 2] + c_
        bound = 32 * 2.0 ** -24 * (f_ * mag[..., m] / np.abs(q[..., 2])
                                   + f_ * np.abs(q[..., m]) * mag[..., 2] / q[..., 2] ** 2 + c_)
        assert np.all(np.abs(coords[..., m].double().cpu().numpy() - want) <= bound)
    k = (p - 1) // 2
    assert np.array_equal(valid.cpu().numpy().astype(bool), (d > 0) & (q[:, k, k, 2] > 0.1 * d))

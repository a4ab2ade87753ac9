"""dpvba_solve_noalloc on problems that nearly fill its 16 MiB: many held
keyframes whose patches tie a few free ones.  Accepted, and bit for bit what
dpvba_solve returns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _graph(dp, held, patches, n_free, seed=0):
    """`held` keyframes of `patches` patches, each patch seen in two of n_free
    frames; every run of patches reaches them all."""
    rs = np.random.RandomState(seed)
    N, P = held + n_free, held * patches
    owner = np.arange(P) // patches
    a = np.arange(P) % n_free
    kk = np.repeat(np.arange(P), 2)
    jj = held + np.stack([a, (a + 1 + rs.randint(0, n_free - 1, P)) % n_free], 1).ravel()
    centre = rs.uniform(-0.3, 0.3, (N, 3))
    uv = np.stack([rs.uniform(60, 580, P), rs.uniform(60, 420, P)], 1)
    d = rs.uniform(0.3, 1.0, P)
    X = np.concatenate([(uv - [320, 240]) / 320, np.ones((P, 1))], 1) / d[:, None] + centre[owner]
    Y = X[kk] - centre[jj]
    target = 320 * Y[:, :2] / Y[:, 2:] + [320, 240] + 0.5 * rs.normal(size=(2 * P, 2))
    grid = np.stack(np.meshgrid([-1.0, 0.0, 1.0], [-1.0, 0.0, 1.0]), -1)
    poses = np.zeros((N, 7))
    poses[:, 6] = 1.0
    poses[:, :3] = centre
    poses[held:, :3] += 0.01 * rs.normal(size=(n_free, 3))
    g = dp.GraphTensors.from_arrays(N, held, uv[:, None, None, :] + grid, owner[kk], jj, kk, target,
                                    rs.uniform(0.1, 1.0, (2 * P, 2)), (320.0, 320.0, 320.0, 240.0))
    return g, poses, d * np.exp(0.05 * rs.normal(size=P))


# rows of 9 blocks (an even number of 16-wide column tiles): 14.8 MiB and 15.4 MiB; frames one
# patch over a tile, whose full tiles need 14.3 MiB (even ones 19.0) and 15.8 MiB (16.2)
@pytest.mark.parametrize("prec,held,patches,n_free,cap", [
    ("fp32", 464, 96, 9, 0), ("fp64", 510, 32, 9, 32), ("fp32", 260, 97, 15, 0), ("fp64", 259, 33, 15, 0)])
def test_noalloc_reaches_its_array(prec, held, patches, n_free, cap):
    import paper_2408_01654_amd as dp

    P, dt = (dp.FP64, torch.float64) if prec == "fp64" else (dp.FP32, torch.float32)
    g, poses, depth = _graph(dp, held, patches, n_free)
    ctx = dp.Context(0)
    try:
        ctx.analyze(g, tile_patches_fp32=cap, tile_patches_fp64=cap)
        print(f"noalloc reach {prec} {held}x{patches} {ctx.analysis_info(P)}", flush=True)
        out = []
        for noalloc in (True, False):
            p = torch.as_tensor(poses, dtype=dt).cuda()
            d = torch.as_tensor(depth, dtype=dt).cuda()
            rep = ctx.solve(g, p, d, n_iters=2, precision=P, noalloc=noalloc)
            assert rep["status"] == 0 and rep["cost"][2] < 0.1 * rep["cost"][0]
            out.append((p, d, rep["cost"]))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
    finally:
        ctx.close()

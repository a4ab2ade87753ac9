"""Selection of loop targets at the sizes of its candidate list (256 a frame):
integer results against the oracle, exactly."""
import numpy as np
import pytest
import torch

from oracle import proximity

pytestmark = pytest.mark.gpu


# every later frame is a candidate: frame 0 has n - 1 of them
@pytest.mark.parametrize("n,max_targets", [(2, 1), (65, 32), (256, 10), (257, 32), (258, 32), (600, 10)])
def test_candidate_list_edges(n, max_targets):
    import paper_2408_01654_amd as dp

    rng = np.random.default_rng(n)
    poses = np.zeros((n, 7), dtype=np.float32)
    poses[:, :3] = rng.uniform(-1, 1, size=(n, 3)).astype(np.float32)
    poses[::7, :3] = poses[0, :3]  # exact ties
    poses[:, 6] = 1.0
    off = np.arange(0, 2 * n + 1, 2).astype(np.int32)
    ctx = dp.Context(0)
    try:
        print(f"proximity list n={n} k={max_targets}", flush=True)
        counts, targets, _, ii, jj, kk = ctx.proximity_edges(torch.as_tensor(poses).cuda(), torch.as_tensor(off).cuda(),
                                                             0, 0, 10.0, max_targets)
        want = proximity.loop_targets(poses[:, :3], 0, 0, 10.0, max_targets)
        got = targets.cpu().numpy()
        assert counts.cpu().tolist() == [len(t) for t in want]
        for i, t in enumerate(want):
            assert got[i, :len(t)].tolist() == t and np.all(got[i, len(t):] == -1), i
        wi, wj, wk = proximity.loop_edges(want, off)
        assert np.array_equal(ii.cpu().numpy(), wi) and np.array_equal(jj.cpu().numpy(), wj)
        assert np.array_equal(kk.cpu().numpy(), wk)
    finally:
        ctx.close()

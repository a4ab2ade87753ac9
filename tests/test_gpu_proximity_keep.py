"""Loop targets of frames with many more candidates than targets: both sides of
where the selection changes (ranks, the last key kept, rounds beyond the list,
the first of which is the candidates' own pass), with exact ties."""
import numpy as np
import pytest
import torch

from oracle import proximity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,max_targets", [(9, 1), (10, 1), (81, 10), (82, 10), (257, 1), (258, 1), (700, 1), (700, 2),
                                           (300, 0)])
def test_kept_targets(n, max_targets):
    import paper_2408_01654_amd as dp

    rng = np.random.default_rng(n + max_targets)
    poses = np.zeros((n, 7), dtype=np.float32)
    poses[:, :3] = rng.uniform(-1, 1, size=(n, 3)).astype(np.float32)
    poses[::5, :3] = poses[0, :3]  # exact ties, at distance zero
    poses[:, 6] = 1.0
    off = np.arange(n + 1).astype(np.int32)
    ctx = dp.Context(0)
    try:
        print(f"proximity kept n={n} k={max_targets}", flush=True)
        counts, targets, _, ii, jj, kk = ctx.proximity_edges(torch.as_tensor(poses).cuda(), torch.as_tensor(off).cuda(),
                                                             0, 0, 10.0, max_targets)
        want = proximity.loop_targets(poses[:, :3], 0, 0, 10.0, max_targets)
        assert counts.cpu().tolist() == [len(t) for t in want]
        got = targets.cpu().numpy()
        assert all(got[i, :len(t)].tolist() == t and np.all(got[i, len(t):] == -1) for i, t in enumerate(want))
        wi, wj, wk = proximity.loop_edges(want, off)
        assert np.array_equal(ii.cpu().numpy(), wi) and np.array_equal(jj.cpu().numpy(), wj)
        assert np.array_equal(kk.cpu().numpy(), wk)
    finally:
        ctx.close()

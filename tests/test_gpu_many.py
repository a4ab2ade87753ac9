"""Several small problems in shared launches (dpvba_solve_many) against each
problem's own call: the same kernels over the same sums, so bit for bit."""
import pytest
import torch

from scenes import tiny_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2408_01654_amd as mod

    return mod


# (n problems, frames of the last): a group of two, one problem beyond a group
# of eight, three groups, and a large problem among small ones (the general way)
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,last,n_iters", [(2, 5, 1), (9, 17, 2), (20, 8, 3), (3, 52, 2)])
def test_many_small_problems_match_one_by_one(dp, prec, n, last, n_iters):
    P = dp.FP64 if prec == "fp64" else dp.FP32
    dt = torch.float64 if prec == "fp64" else torch.float32
    scenes = [tiny_scene(3 + (5 * i) % 15, 4 + (7 * i) % 40, seed=i) for i in range(n - 1)]
    scenes.append(tiny_scene(last, 12, seed=4, radius=5, trajectory="forward"))
    ctxs = [dp.Context(0) for _ in scenes]
    try:
        gs = [dp.GraphTensors.from_scene(s) for s in scenes]
        for c, g in zip(ctxs, gs):
            c.analyze(g)
        p0 = [torch.as_tensor(s.poses, dtype=dt).cuda().contiguous() for s in scenes]
        d0 = [torch.as_tensor(s.inv_depth, dtype=dt).cuda().contiguous() for s in scenes]
        kw = dict(n_iters=n_iters, lam=1e-4, z_min=0.1, precision=P)
        for _ in range(2):  # twice: the contexts' barrier slots alternate
            pm, dm = [p.clone() for p in p0], [d.clone() for d in d0]
            print(f"many {prec} n={n} last={last}", flush=True)
            dp.solve_many(ctxs, gs, pm, dm, **kw)
            torch.cuda.synchronize()
            for i, (c, g) in enumerate(zip(ctxs, gs)):
                p1, d1 = p0[i].clone(), d0[i].clone()
                c.solve(g, p1, d1, report=False, **kw)
                torch.cuda.synchronize()
                assert torch.isfinite(p1).all() and not torch.equal(p1, p0[i])
                assert torch.equal(pm[i], p1) and torch.equal(dm[i], d1)
    finally:
        for c in ctxs:
            c.close()

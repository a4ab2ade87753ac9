"""Calls over many small problems: launches that hold more workgroups than the
device does at once, a captured call with a problem that loses its steps, and
adjoints in several groups of very different windows, some without one of the
gradients.  Each problem as by its own call, bit for bit (the same kernels over
the same sums)."""
import dataclasses

import pytest
import torch

from scenes import tiny_scene

pytestmark = pytest.mark.gpu


def _problems(dp, scenes, dt):
    ctxs = [dp.Context(0) for _ in scenes]
    gs = [dp.GraphTensors.from_scene(s) for s in scenes]
    for c, g in zip(ctxs, gs):
        c.analyze(g)
    return (ctxs, gs, [torch.as_tensor(s.poses, dtype=dt).cuda() for s in scenes],
            [torch.as_tensor(s.inv_depth, dtype=dt).cuda() for s in scenes])


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_more_workgroups_than_the_device_holds(prec):
    import paper_2408_01654_amd as dp

    P, dt = (dp.FP64, torch.float64) if prec == "fp64" else (dp.FP32, torch.float32)
    scenes = [tiny_scene(120 + 7 * i, 2 + i, seed=i, radius=3, n_fixed=108 + 7 * i, trajectory="forward")
              for i in range(5)]
    ctxs, gs, p0, d0 = _problems(dp, scenes, dt)
    try:
        for n_iters in (1, 3):
            kw = dict(n_iters=n_iters, lam=1e-4, z_min=0.1, precision=P)
            p, d = [x.clone() for x in p0], [x.clone() for x in d0]
            print(f"wide groups {prec} {n_iters}", flush=True)
            dp.solve_many(ctxs, gs, p, d, **kw)
            for i, (c, g) in enumerate(zip(ctxs, gs)):
                q, e = p0[i].clone(), d0[i].clone()
                c.solve(g, q, e, report=False, **kw)
                assert torch.isfinite(q).all() and not torch.equal(q, p0[i])
                assert torch.equal(p[i], q) and torch.equal(d[i], e)
    finally:
        for c in ctxs:
            c.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_lost_steps_in_a_captured_group(prec):
    """Undamped, a pose without an edge leaves a zero pivot: that problem's
    steps are discarded, the others' are not."""
    import paper_2408_01654_amd as dp

    P, dt = (dp.FP64, torch.float64) if prec == "fp64" else (dp.FP32, torch.float32)
    scenes = [tiny_scene(4 + 3 * i, 9, seed=i) for i in range(4)]
    s = scenes[1]
    keep = (s.ii != s.n_frames - 1) & (s.jj != s.n_frames - 1)
    scenes[1] = dataclasses.replace(s, ii=s.ii[keep], jj=s.jj[keep], kk=s.kk[keep], target=s.target[keep],
                                    weight=s.weight[keep], patches=s.patches[:-9], inv_depth=s.inv_depth[:-9])
    ctxs, gs, p0, d0 = _problems(dp, scenes, dt)
    kw = dict(n_iters=3, lam=0.0, z_min=0.1, precision=P)
    try:
        print(f"lost steps {prec}", flush=True)
        ref = [(p.clone(), d.clone()) for p, d in zip(p0, d0)]
        for c, g, (q, e) in zip(ctxs, gs, ref):
            c.solve(g, q, e, report=False, **kw)
        for i, (q, e) in enumerate(ref):
            assert torch.isfinite(q).all() and torch.equal(q, p0[i]) == torch.equal(e, d0[i]) == (i == 1)
        p, d = [x.clone() for x in p0], [x.clone() for x in d0]
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            dp.solve_many(ctxs, gs, p, d, **kw)
        for _ in range(3):
            for x, y in zip(p + d, p0 + d0):
                x.copy_(y)
            graph.replay()
            torch.cuda.synchronize()
            for i, (q, e) in enumerate(ref):
                assert torch.equal(p[i], q) and torch.equal(d[i], e)
    finally:
        torch.cuda.synchronize()
        for c in ctxs:
            c.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [7, 13, 16])
def test_adjoints_in_several_groups(prec, n):
    import paper_2408_01654_amd as dp

    P, dt = (dp.FP64, torch.float64) if prec == "fp64" else (dp.FP32, torch.float32)
    scenes = [tiny_scene(3 + (5 * i) % 15, 3 + (17 * i) % 61, seed=i, radius=3 + i % 6, trajectory="forward")
              for i in range(n)]
    ctxs, gs, p0, d0 = _problems(dp, scenes, dt)
    try:
        gen = torch.Generator().manual_seed(n)
        up = lambda x: torch.randn(x.shape, generator=gen, dtype=dt).cuda()
        gp = [None if i % 4 == 1 else up(x) for i, x in enumerate(p0)]
        gd = [None if i % 3 == 1 else up(x) for i, x in enumerate(d0)]
        kw = dict(n_iters=2, lam=1e-4, z_min=0.1, precision=P)
        print(f"adjoint groups {prec} {n}", flush=True)
        gt, gw = dp.solve_backward_many(ctxs, gs, p0, d0, gp, gd, **kw)
        torch.cuda.synchronize()
        for i, (c, g) in enumerate(zip(ctxs, gs)):
            t, w = c.solve_backward(g, p0[i], d0[i], gp[i], gd[i], **kw)
            assert torch.isfinite(t).all() and torch.isfinite(w).all()
            assert torch.equal(gt[i], t) and torch.equal(gw[i], w)
    finally:
        for c in ctxs:
            c.close()

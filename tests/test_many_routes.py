"""Which problems of a bundle_adjust_many share launches and which are solved
in turn, on the host with stand-in contexts."""
import pytest
import torch

import paper_2408_01654_amd as dp
from paper_2408_01654_amd import binding


class _Ctx:
    def __init__(self, log, device=0, tracing=False):
        self.log, self.device, self.tracing = log, device, tracing

    def solve(self, g, poses, inv_depth, n_iters, lam, z_min, precision, report):
        self.log.append(("one", self))


def _graph(frames, fixed, edges=4):
    z = torch.zeros(edges, dtype=torch.int32)
    return dp.GraphTensors(frames, fixed, torch.zeros(2, 1, 1, 2), z, z, z, torch.zeros(edges, 2),
                           torch.zeros(edges, 2), (1.0, 1.0, 0.0, 0.0))


SMALL, FREELESS, EDGELESS, LARGE = (8, 2), (8, 8), (8, 2, 0), (20, 2)


@pytest.mark.parametrize("shapes,kw,shared", [
    ([SMALL] * 3, {}, [0, 1, 2]),
    ([SMALL, FREELESS, SMALL], {}, [0, 2]),           # no free pose: in turn, the others still share
    ([SMALL, SMALL, EDGELESS], {}, [0, 1]),
    ([SMALL, LARGE, SMALL, LARGE], {}, [0, 2]),
    ([SMALL, LARGE], {}, []),                          # one alone is its own launch
    ([SMALL, SMALL], {"n_iters": 0}, []),
    ([SMALL, SMALL], {"precision": dp.MIXED}, []),
    ([SMALL, SMALL], {"devices": [0, 1]}, []),         # contexts of two devices
    ([SMALL, SMALL, SMALL], {"traced": [1]}, [0, 2]),  # a traced context's phases are its own
    ([SMALL, SMALL], {"same": True}, []),
])
def test_forward_routes(monkeypatch, shapes, kw, shared):
    log = []
    monkeypatch.setattr(binding, "solve_many", lambda cs, gs, p, d, *a, **k: log.append(("many", list(cs))))
    devices, traced = kw.get("devices", [0] * len(shapes)), kw.get("traced", [])
    ctxs = [_Ctx(log, devices[i], i in traced) for i in range(len(shapes))]
    if kw.get("same"):
        ctxs = ctxs[:1] * len(shapes)
    gs = [_graph(*s) for s in shapes]
    p0 = [torch.zeros(g.n_frames, 7) for g in gs]
    d0 = [torch.zeros(2) for _ in gs]
    with torch.no_grad():
        dp.bundle_adjust_many(ctxs, gs, p0, d0, [g.target for g in gs], [g.weight for g in gs],
                              n_iters=kw.get("n_iters", 2), precision=kw.get("precision", dp.FP32))
    many = [x for kind, x in log if kind == "many"]
    assert many == ([[ctxs[i] for i in shared]] if shared else [])
    assert [x for kind, x in log if kind == "one"] == [c for i, c in enumerate(ctxs) if i not in shared]

"""A forcing call replayed as a graph after ibmx_plan_reserve has moved the
workspace that the captured launches use (the scan of more than 2048 tiles):
the same bits as the eager call."""
import numpy as np
import pytest

from paper_2109_03972_amd import ibmx, synth
from tests._util import require_gpu

pytestmark = pytest.mark.gpu


def test_graph_after_a_growth_of_the_workspace():
    import torch
    dev = require_gpu()
    n = (256, 256, 128)                      # 4096 tiles of 16 x 16 x 8
    rng = np.random.default_rng(4)
    d = np.full(60, 10.0)
    moff, body, dV = synth.build_markers(d, 1.0, rng)
    prm = dict(synth.default_params(), disable_mode=0, n_iter=2)
    plan = ibmx.Plan(n, 1.0, (0.0, 0.0, 0.0), (1, 1, 1), prm, moff, "f32")
    assert plan.stats()["tiles"] > 2048

    def t(a):
        return torch.as_tensor(a, dtype=torch.float64, device=dev).contiguous()

    keep = t(body), t(dV)
    plan.set_markers(*keep)
    x = t(rng.random((3, 60)) * np.array(n)[:, None])
    up, wp = t(rng.normal(0, 0.1, (3, 60))), t(rng.normal(0, 0.05, (3, 60)))
    u0 = torch.randn((3, 128, 256, 256), device=dev)
    u, f = u0.clone(), torch.zeros_like(u0)
    S, T = torch.zeros_like(x), torch.zeros_like(x)

    def call(graph):
        u.copy_(u0)
        f.zero_()
        plan.forcing(u, f, x, up, wp, S=S, T=T, graph=graph)
        plan.check("forcing")
        return [v.clone() for v in (u, f, S, T)]

    want = call(False)
    for cells in (0, 100_000, 1_000_000):
        if cells:
            plan.reserve(cell_cap=cells)
        for _ in range(3):
            for a, b in zip(call(True), want):
                assert torch.equal(a, b), cells
    plan.close()

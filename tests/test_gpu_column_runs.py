"""Length of the stencil kernels' runs along z: FP32 and FP64 plans split the
same grid differently (32 to 4 planes; a last run of one plane, a column shorter
than a run) and compute the same FP64 arithmetic, so the FP32 plan's predictor
holds the FP64 plan's values rounded once (half a unit in the last place, one
allowed)."""
import numpy as np
import pytest

from paper_2109_03972_amd import ibmx, synth
from tests._util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(256, 256, 33), (150, 133, 177), (64, 64, 130), (64, 16, 3),
                               (70, 9, 257)])
@pytest.mark.parametrize("periodic", [(1, 1, 0), (0, 1, 0)])
def test_predictor_runs(n, periodic):
    import torch
    dev = require_gpu()
    g = torch.Generator(device=dev).manual_seed(1)
    shape = (n[2], n[1], n[0])
    u, N, P = (torch.randn(k + shape, generator=g, device=dev, dtype=torch.float32)
               for k in ((3,), (3,), ()))
    prm = dict(synth.default_params(), disable_mode=0)
    out = {}
    for prec, T in (("f32", torch.float32), ("f64", torch.float64)):
        plan = ibmx.Plan(n, 1.0, (0.0, 0.0, 0.0), periodic, prm, np.zeros(1, np.int32), prec)
        Nb = N.to(T).clone()
        ut, lap = plan.fluid_predictor(u.to(T).contiguous(), Nb, P.to(T).contiguous(), 0.5, 0.4,
                                       -0.3)
        plan.check("predictor")
        plan.close()
        out[prec] = [v.double().cpu().numpy() for v in (ut, Nb, lap)]
    for a, b in zip(out["f32"], out["f64"]):
        assert np.all(np.abs(a - b) <= np.abs(b) * 2.0 ** -23 + 1e-30)

"""The default tiles follow the delta: a plan moved to the other one by
set_params has the shape that a plan created with it has, unless a shape was
chosen; results against the oracle each way (tolerances as for every forcing
output)."""
import numpy as np
import pytest

import oracle
from paper_2109_03972_amd import ibmx, synth
from tests._util import gpu_forcing, rel_err, require_gpu

pytestmark = pytest.mark.gpu

SHAPE = {("f64", 3): (16, 16, 8), ("f64", 4): (16, 8, 8), ("f32", 3): (16, 16, 8),
         ("f32", 4): (16, 16, 8)}


@pytest.mark.parametrize("n", [(48, 40, 48), (40, 33, 21)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("first", [3, 4])
def test_default_tiles_follow_the_delta(first, precision, n):
    import torch
    dev = require_gpu()
    case = synth.small_case(77, n=n, periodic=(1, 1, 1), diameters=(6.0,), n_iter=2,
                            disable_mode=0)
    prm = {k: dict(case.params, kernel=k, eps_sep=2.0, lub_C=4.0, gap_cut=4.0) for k in (3, 4)}
    plan = ibmx.Plan.from_case(case, precision, params=prm[first])
    keep = [torch.as_tensor(v, device=dev).contiguous() for v in (case.body, case.dV)]
    plan.set_markers(*keep)
    fresh = {}
    for k in (first, 7 - first, first):
        plan.set_params(prm[k])
        other = ibmx.Plan.from_case(case, precision, params=prm[k])
        want = other.stats()["tile"]
        other.close()
        if n[1] == 40:
            assert want == SHAPE[precision, k]
        assert plan.stats()["tile"] == want
        ref = oracle.forcing(case, kernel=k)
        got = gpu_forcing(case, precision, params=prm[k], plan=plan)
        for q in ("u", "f_tot", "S", "T"):
            e = rel_err(got[q], ref[q])
            assert e <= (1e-12 if precision == "f64" else 1e-4), f"{k} {q}: {e:.2e}"
        if k in fresh:
            for q in ("u", "f_tot"):
                np.testing.assert_array_equal(got[q], fresh[k][q])
        fresh[k] = got
    plan.set_tiles(8, 8, 8)
    chosen = plan.stats()["tile"]
    plan.set_params(prm[7 - first])
    assert plan.stats()["tile"] == chosen
    plan.close()

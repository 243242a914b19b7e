"""The pair search where it changes: partners kept by the search or searched
again (32 per particle), walls of every side, dense and single cells, centres
on the domain's edges and whole periods away (the wrap's fast path); lists, gaps
and forces against the oracle as everywhere in the pair pass."""
import numpy as np
import pytest

import oracle
from paper_2109_03972_amd import synth
from tests.test_gpu_pairs import _check, _gpu_pairs

pytestmark = pytest.mark.gpu


def _spheres(x, R, periodic, n=(48, 40, 44)):
    case = synth.small_case(3, n=n, periodic=periodic, diameters=(6.0,), disable_mode=0)
    rng = np.random.default_rng(1)
    k = len(R)
    case.xp, case.radius, case.mass = np.ascontiguousarray(x), np.asarray(R), np.ones(k)
    case.up, case.wp = rng.normal(0.0, 0.1, (3, k)), rng.normal(0.0, 0.05, (3, k))
    case.moff, case.body, case.dV = np.zeros(k + 1, np.int32), np.zeros((3, 0)), np.ones(k)
    return case


@pytest.mark.parametrize("around", [31, 32, 33, 64, 65, 150])
def test_partners_kept_and_searched_again(around):
    p = synth.spiral_points(around).T * (8.0 + 1.2)     # gap 0.2 to the big one
    rng = np.random.default_rng(around)
    x = np.concatenate([[[24.0], [20.0], [22.0]], p + np.array([[24.0], [20.0], [22.0]])], 1)
    x[:, 1:] = x[:, 1 + rng.permutation(around)]
    case = _spheres(x, [8.0] + [1.0] * around, (1, 1, 1))
    ref, _ = _check(case, _gpu_pairs(case))
    assert (ref["pairs"][0] == 0).sum() == around


@pytest.mark.parametrize("periodic", [(1, 1, 1), (0, 0, 0), (1, 0, 1)])
@pytest.mark.parametrize("rmax", [0.7, 30.0])
def test_edges_seams_and_walls(periodic, rmax):
    """Random small spheres, some with coordinates exactly on the domain's ends,
    one unit in the last place off them, or (periodic) whole periods away; with
    the large bound all share one cell."""
    rng = np.random.default_rng(5)
    n, k = (48, 40, 44), 300
    x = rng.random((3, k)) * np.array(n)[:, None]
    for a in range(3):
        L = float(n[a])
        for q, v in enumerate((0.0, L, np.nextafter(L, 0.0), np.nextafter(0.0, 1.0), 0.5 * L)):
            x[a, 10 * a + q] = v
        if periodic[a]:
            x[a, 40 + a] += L
            x[a, 50 + a] -= 3 * L
            x[a, 60 + a] = -1e-17
    case = _spheres(x, rng.uniform(0.4, 0.7, k), periodic)
    if rmax > 1.0:
        # one cell per axis: a large sphere that touches none but widens the bound
        case.radius[0], case.xp[:, 0] = 15.0, 21.0
    _check(case, _gpu_pairs(case))


@pytest.mark.parametrize("around", [20, 32, 33, 64, 150])
@pytest.mark.parametrize("short", [1, 7, 19])
def test_short_lists_hold_the_first_pairs(around, short):
    """A capacity that cuts the list within one particle's partners: the entries
    that fit are the first of the canonical order, whichever way the partners
    were found."""
    import torch
    from paper_2109_03972_amd import ibmx
    from tests._util import dev_case
    p = synth.spiral_points(around).T * (8.0 + 1.2)
    rng = np.random.default_rng(around)
    x = np.concatenate([[[24.0], [20.0], [22.0]], p + np.array([[24.0], [20.0], [22.0]])], 1)
    x[:, 1:] = x[:, 1 + rng.permutation(around)]
    case = _spheres(x, [8.0] + [1.0] * around, (1, 1, 1))
    case.u0 = None
    ref = oracle.pairs(case)
    D = dev_case(case, "f64")
    plan = ibmx.Plan.from_case(case, "f64")
    plan.set_markers(D["body"], D["dV"])
    for cap in (around - short, around - 1, around):
        res = plan.pairs(D["xp"], D["radius"], D["mass"], D["up"], D["wp"], pair_cap=cap)
        over = cap < ref["pairs"].shape[1]
        assert plan.status() == (ibmx.ECAPACITY if over else ibmx.OK)
        assert int(res["counts"][0]) == ref["pairs"].shape[1]
        k = min(cap, ref["pairs"].shape[1])
        np.testing.assert_array_equal(res["pairs"][:, :k].cpu().numpy(), ref["pairs"][:, :k])
        np.testing.assert_allclose(res["gap"][:k].cpu().numpy(), ref["gap"][:k], rtol=0, atol=1e-12)
    plan.close()

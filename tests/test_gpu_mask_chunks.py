"""The marker mask of a particle with more close pairs than the kernel takes at
a time (64 of its partners and walls): later chunks may only clear markers, in
both disable modes, and the walls come last; bit for bit with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2109_03972_amd import synth
from tests.test_gpu_pairs import _check, _gpu_pairs

pytestmark = pytest.mark.gpu


def _crowd(around, mode, seed, close_last):
    """A sphere of 16 cells by the lower wall among small ones: gaps of 0.2
    (its or their markers drop) and 4.5 (listed only)."""
    rng = np.random.default_rng(around)
    p = synth.spiral_points(2 * around).T
    p = p[:, p[2] > -0.7][:, :around]
    assert p.shape[1] == around
    gap = np.where(np.arange(around) % 3 == 1, 4.5, 0.2)
    if close_last:                      # the first chunk drops nothing
        gap = np.where(np.arange(around) < 64, 4.5, 0.2)
    d = np.concatenate([[16.0], np.full(around, 1.6)])
    x = np.empty((3, around + 1))
    x[:, 0] = 33.0, 30.0, 8.9
    x[:, 1:] = x[:, :1] + p * (8.0 + 0.8 + gap)
    case = synth.small_case(3, n=(66, 64, 48), periodic=(1, 1, 0), diameters=(6.0,))
    case.xp, case.radius, case.mass = x, 0.5 * d, np.ones(around + 1)
    case.up, case.wp = rng.normal(0.0, 0.1, x.shape), rng.normal(0.0, 0.05, x.shape)
    case.moff, case.body, case.dV = synth.build_markers(d, 1.0, rng)
    case.u0 = None
    case.params = dict(case.params, gap_cut=6.0, disable_mode=mode, disable_seed=seed)
    return case


@pytest.mark.parametrize("seed", [7, 8])
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("around,close_last", [(63, False), (64, False), (65, False),
                                               (150, False), (150, True)])
def test_mask_of_a_crowded_particle(around, mode, seed, close_last):
    case = _crowd(around, mode, seed, close_last)
    ref, _ = _check(case, _gpu_pairs(case))
    mine = ref["pairs"][0] == 0
    assert mine.sum() == around and np.any(ref["walls"][0] == 0)
    # what the first 64 entries alone would give differs
    short = {k: (v[..., ~(mine & (np.cumsum(mine) > 64))] if k in ("pairs", "gap") else v)
             for k, v in ref.items()}
    if around >= 64:
        for k in ("walls", "wgap"):
            short[k] = short[k][..., ref["walls"][0] != 0]
    full, cut = oracle.marker_mask(case, ref), oracle.marker_mask(case, short)
    assert 0 < full.sum() < full.size
    if around >= 64 and (mode == 1 or close_last):
        assert np.any(full != cut)

"""Particle integrals at the edges of their inputs: field values that must not
count, particles that are nowhere, boxes longer than 16 bits, wide spheres
among many; and the rounding of the sums."""
import numpy as np
import pytest

import oracle
from paper_2109_03972_amd import ibmx, synth
from tests._util import rel_err, require_gpu

pytestmark = pytest.mark.gpu


def _spheres(n, x, R, periodic=(1, 1, 0), seed=5):
    case = synth.small_case(seed, n=n, periodic=periodic, diameters=(6.0,), disable_mode=0)
    k = len(R)
    case.xp, case.radius, case.mass = np.ascontiguousarray(x), np.asarray(R), np.ones(k)
    case.up, case.wp = np.zeros((3, k)), np.zeros((3, k))
    case.moff, case.body, case.dV = np.zeros(k + 1, np.int32), np.zeros((3, 0)), np.ones(k)
    return case


def _integrals(case, u, precision="f64"):
    import torch
    dev = require_gpu()
    T = torch.float64 if precision == "f64" else torch.float32
    plan = ibmx.Plan.from_case(case, precision)
    x, R = (torch.as_tensor(a, device=dev).contiguous() for a in (case.xp, case.radius))
    Iu, Ir = plan.particle_integrals(torch.as_tensor(u, device=dev).to(T).contiguous(), x, R)
    plan.check("integrals")
    plan.close()
    return Iu.cpu().numpy(), Ir.cpu().numpy()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("count", [3, 600, 4200])
def test_values_outside_the_particles_do_not_count(count, bad):
    """A NaN or an infinity in every cell of volume fraction 0: the sums are
    those of a field with 0 there, bit for bit (such a cell is left out)."""
    n = (72, 64, 80)
    rng = np.random.default_rng(count)
    x = rng.random((3, count)) * np.array(n)[:, None]
    case = _spheres(n, x, rng.uniform(0.7, 2.5 if count > 100 else 9.0, count))
    alpha = oracle.particle_integrals(case, u=case.u0, want_alpha=True)["alpha"]
    out = alpha == 0.0
    assert 0.05 < out.mean() < 1.0
    want = _integrals(case, np.where(out, 0.0, case.u0))
    got = _integrals(case, np.where(out, bad, case.u0))
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("what", ["centre", "radius"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("count", [4, 600, 4200])
def test_particles_that_are_not_finite(count, bad, what):
    """A particle whose centre or radius is not finite has no cells: its sums
    are 0, the others' as without it, and a call in which every particle is
    lost takes no longer than one with small spheres (a walk of this grid by
    every one took 290 times as long)."""
    import torch
    dev = require_gpu()
    n = (256, 256, 256)
    rng = np.random.default_rng(count)
    x, R = rng.random((3, count)) * 256.0, rng.uniform(0.7, 2.5, count)
    case = _spheres(n, x, R)
    u = torch.rand((3, 256, 256, 256), dtype=torch.float32, device=dev)
    plan = ibmx.Plan.from_case(case, "f32")

    def call(x, R, reps=0):
        X, Q = (torch.as_tensor(a, device=dev).contiguous() for a in (x, R))
        out = plan.particle_integrals(u, X, Q)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(reps):
            plan.particle_integrals(u, X, Q)
        b.record()
        torch.cuda.synchronize()
        return [v.cpu().numpy() for v in out], a.elapsed_time(b)

    def lose(which):
        xb, Rb = x.copy(), R.copy()
        if what == "radius":
            Rb[which] = bad
        else:
            xb[rng.integers(0, 3, len(which)), which] = bad
        return xb, Rb

    want, t0 = call(x, R, 10)
    lost = np.array([1, count - 1])
    got, _ = call(*lose(lost))
    for a, b in zip(got, want):
        assert np.all(a[:, lost] == 0.0)
        np.testing.assert_array_equal(np.delete(a, lost, 1), np.delete(b, lost, 1))
    got, t1 = call(*lose(np.arange(count)), 10)
    assert all(np.all(a == 0.0) for a in got)
    assert t1 <= 4.0 * t0, (t1, t0)
    plan.close()


def _plain_integrals(n, x, R, u):
    """The level-set sums over every cell of a walled box, h = 1."""
    i = [np.arange(m) - c for m, c in zip(n, x)]
    num = den = 0.0
    for m in range(8):
        d2 = ((i[2] + (m >> 2)) ** 2)[:, None, None] + \
            ((i[1] + (m >> 1 & 1)) ** 2)[None, :, None] + ((i[0] + (m & 1)) ** 2)[None, None, :]
        phi = np.sqrt(d2) - R
        num, den = num + np.maximum(-phi, 0.0), den + np.abs(phi)
    w = num / den * u
    r = [(i[2 - a] + 0.5).reshape([-1 if b == a else 1 for b in range(3)]) for a in (2, 1, 0)]
    Ir = [(r[1] * w[2] - r[2] * w[1]).sum(), (r[2] * w[0] - r[0] * w[2]).sum(),
          (r[0] * w[1] - r[1] * w[0]).sum()]
    return w.sum((1, 2, 3)), np.array(Ir)


@pytest.mark.parametrize("n", [(80000, 5, 4), (5, 80000, 4), (4, 5, 80000)])
def test_boxes_longer_than_16_bits(n):
    """A sphere whose box is 78001 cells long, cut by the lower wall; sums of
    1.6M values of one sign to FP64 rounding (1e-12)."""
    rng = np.random.default_rng(1)
    a = int(np.argmax(n))
    x = 0.5 * np.array(n) + 0.13
    x[a] = 38000.3
    u = 1.0 + rng.random((3, n[2], n[1], n[0]))
    case = synth.Case(name="long", n=n, h=1.0, origin=(0.0, 0.0, 0.0), periodic=(0, 0, 0),
                      xp=x[:, None].copy(), up=np.zeros((3, 1)), wp=np.zeros((3, 1)),
                      radius=np.array([40000.0]), mass=np.ones(1),
                      moff=np.zeros(2, np.int32), body=np.zeros((3, 0)), dV=np.ones(1), u0=u,
                      params=dict(synth.default_params(), disable_mode=0))
    for got, want in zip(_integrals(case, u), _plain_integrals(n, x, 40000.0, u)):
        assert rel_err(got[:, 0], want) <= 1e-12


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("count", [256, 257, 1535, 1536, 4095, 4096, 4101])
def test_wide_spheres_among_many(count, precision):
    """Spheres about the widths (10 and 40 cells) from which a workgroup takes
    one, several of a group of four, across seams, the last ones, in every split
    of particles over waves: against the
    oracle as everywhere (FP64 sums in another order, 1e-12; an FP32 field
    holds what the oracle reads)."""
    n = (150, 80, 160)
    rng = np.random.default_rng(count)
    x, R = rng.random((3, count)) * np.array(n)[:, None], rng.uniform(0.6, 2.5, count)
    R[[0, 1, 3, 5, 10]] = 36.4, 19.9, 30.0, np.nextafter(20.0, 30.0), 20.0
    R[[20, 21, 22]] = 5.0, np.nextafter(5.0, 6.0), 7.0
    R[count - 2:] = 25.0, 21.0
    x[:, 0], x[:, 3] = (3.2, 19.0, 70.0), (140.1, 79.7, 2.5)
    case = _spheres(n, x, R)
    u = case.u0.astype(np.float32).astype(np.float64)
    ref = oracle.particle_integrals(case, u=u)
    for k, got in zip(("Iu", "Ir"), _integrals(case, u, precision)):
        assert rel_err(got, ref[k]) <= 1e-12, k


@pytest.mark.parametrize("count,R,which,bound", [(240, (8.0, 12.0), 0, 0.82),
                                                 (4100, (12.0, 12.0), 1, 0.143)])
def test_rounding_of_the_sums(count, R, which, bound):
    """RMS error over 150 spheres against 80-bit sums, in units of 2^-53 of the
    sum of the terms' sizes.  An addition rounds by 0.43 units of its result (rms
    over the results' mantissas), so a tree over 16 waves of 64 lanes by sqrt(2)
    of that, 0.61 of the sum, where adding the waves in turn takes 1.0: sixteen
    waves per sphere, Iu, bound 0.82.  One wave per sphere, Ir: a lane's 113
    inside cells in one chain drift with the mean velocity, 0.2; in blocks of 16
    0.06, and 0.04 from the surface cells: bound 0.143."""
    L = np.longdouble
    n = (96, 96, 96)
    rng = np.random.default_rng(count)
    x, rad = rng.random((3, count)) * 96.0, rng.uniform(*R, count)
    u = rng.uniform(1.2, 1.4, (3, 96, 96, 96))
    case = _spheres(n, x, rad, periodic=(1, 1, 1))
    got = _integrals(case, u)[which]
    err = []
    for p in range(150):
        lo = np.floor(x[:, p] - rad[p]).astype(int)
        ax = [np.arange(lo[a], int(np.floor(x[a, p] + rad[p])) + 1) for a in range(3)]
        i = [(ax[a] - x[a, p].astype(L)).reshape([-1 if b == 2 - a else 1 for b in range(3)])
             for a in range(3)]
        num = den = L(0)
        for m in range(8):
            phi = np.sqrt((i[0] + (m & 1)) ** 2 + (i[1] + (m >> 1 & 1)) ** 2 +
                          (i[2] + (m >> 2)) ** 2) - L(rad[p])
            num, den = num + np.maximum(-phi, 0), den + np.abs(phi)
        w = num / den * u[(slice(None), *np.ix_(ax[2] % 96, ax[1] % 96, ax[0] % 96))]
        r = [v + L(0.5) for v in i]
        terms = w if which == 0 else np.stack([r[1] * w[2] - r[2] * w[1],
                                               r[2] * w[0] - r[0] * w[2],
                                               r[0] * w[1] - r[1] * w[0]])
        err.append((got[:, p] - terms.sum((1, 2, 3))) / np.abs(terms).sum((1, 2, 3)))
    rms = float(np.sqrt(np.mean(np.square(err)))) * 2.0 ** 53
    print(f"{count} {rms:.3f}", flush=True)
    assert rms <= bound

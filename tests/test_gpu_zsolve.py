"""The solve along z of the fluid steps at the column lengths where its
split changes (rows per thread, waves per column, front padding), with walls
and periodic, and the systems that keep the elimination or the FFT along z (a
negative or very large viscous number, columns over 2048 rows), against the
FP64 oracle.

Tolerance 1e-12 in FP64: the filters lose about 1/sqrt(eps) roundings in a
mode, eps its distance from the singular system (3.8e-5 at 1024 points,
4e-2 here), below the elimination's own 1e-13."""
import numpy as np
import pytest

from oracle import fluid_stage as fs
from oracle import projection as pj
from paper_2109_03972_amd import ibmx
from tests._util import rel_err, require_gpu
from tests.test_gpu_fluid import _case, _run

pytestmark = pytest.mark.gpu

WALLS = [15, 16, 31, 33, 127, 128, 129, 256, 257, 513]


@pytest.mark.parametrize("nz,wall", [(n, 1) for n in WALLS] +
                         [(n, 0) for n in (8, 32, 128, 256, 512, 1024)])
def test_projection_columns(nz, wall):
    n, per = (8, 8, nz), (1, 1, 0 if wall else 1)
    case = _case(n, per, seed=nz)
    rng = np.random.default_rng(nz)
    u0, P0 = rng.normal(0.0, 1.0, (3, nz, 8, 8)), rng.normal(0.0, 1.0, (nz, 8, 8))
    prm = case.params
    ref = pj.project(u0, P0, case.h, prm["c"], prm["nu_f"], 0.0, per)
    got = _run(case, "f64", u0, P0, 0.0)
    for k in ("u", "uf", "P", "phi"):
        assert rel_err(got[k], ref[k]) <= 1e-12, k


@pytest.mark.parametrize("nz", [1025, 2048, 2049])
def test_projection_long_columns(nz):
    """Columns at the end of the range, where the oracle's dense solves take
    too long: the projected faces are divergence-free to the rounding of phi
    (each of the Laplacian's 12 weights 1/h^2, 32 roundings)."""
    n, per = (8, 8, nz), (1, 1, 0)
    case = _case(n, per, seed=nz)
    rng = np.random.default_rng(nz)
    u0, P0 = rng.normal(0.0, 1.0, (3, nz, 8, 8)), rng.normal(0.0, 1.0, (nz, 8, 8))
    got = _run(case, "f64", u0, P0, 0.0)
    tol = 32 * 12 * np.finfo(float).eps * np.abs(got["phi"]).max() * case.params["c"] / case.h ** 3
    assert np.abs(pj.face_div(got["uf"], case.h, per)).max() <= tol
    assert abs(got["phi"].mean()) <= 1e-12 * np.abs(got["phi"]).max()


@pytest.mark.parametrize("nz,wall", [(n, 1) for n in WALLS] + [(n, 0) for n in (8, 64, 256)])
@pytest.mark.parametrize("nu", [0.3, 0.0, -0.1, 1.0e3, 1.0e5])
def test_viscous_columns(nz, wall, nu):
    import torch
    dev = require_gpu()
    n, per = (8, 8, nz), (1, 1, 0 if wall else 1)
    case = _case(n, per, seed=3)
    alpha, dt = 1.0 / 15.0, 0.4
    case.params = dict(case.params, c=2.0 * alpha * dt, nu_f=nu)
    rng = np.random.default_rng(nz)
    shape = (3, nz, n[1], 8)
    u0, lap = rng.normal(size=shape), rng.normal(size=shape)
    P = rng.normal(size=shape[1:])
    ref = fs.helmholtz(u0, lap, P, None, case.h, nu, alpha, 0.0, dt, per)
    plan = ibmx.Plan.from_case(case, "f64")
    u = torch.as_tensor(u0, device=dev).contiguous()
    plan.fluid_helmholtz(u, torch.as_tensor(lap, device=dev), torch.as_tensor(P, device=dev), dt)
    plan.check("helmholtz")
    e = rel_err(u.cpu().numpy(), ref)
    plan.close()
    assert e <= 1e-12, e


@pytest.mark.parametrize("nz,wall", [(64, 1), (300, 1), (64, 0)])
@pytest.mark.parametrize("nu", [5e-324, 1e-310, 1e-307, 1e-200])
def test_vanishing_viscosity(nz, wall, nu):
    """A viscosity too small to couple the rows: the same bits as without any."""
    import torch
    dev = require_gpu()
    n, per = (8, 8, nz), (1, 1, 0 if wall else 1)
    case = _case(n, per, seed=3)
    rng = np.random.default_rng(nz)
    u0, lap = (torch.as_tensor(rng.normal(size=(3, nz, 8, 8)), device=dev) for _ in range(2))
    P = torch.zeros((nz, 8, 8), dtype=torch.float64, device=dev)
    out = []
    for v in (0.0, nu):
        case.params = dict(case.params, c=0.8, nu_f=v)
        plan = ibmx.Plan.from_case(case, "f64")
        u = u0.clone()
        plan.fluid_helmholtz(u, lap, P, 0.4)
        plan.check("helmholtz")
        plan.close()
        out.append(u.cpu().numpy())
    assert np.isfinite(out[0]).all()
    np.testing.assert_array_equal(*out)


@pytest.mark.parametrize("nz", [64, 200])
@pytest.mark.parametrize("beta", [1.0 / 750.0, 2.0 / 15.0])
def test_rounding_of_a_column(nz, beta):
    """RMS error of the viscous columns between walls against an 80-bit
    elimination, in units of 2^-53 of the solution's RMS.  Fields that only
    change sign along x and y have one mode, and their transforms are exact.  A
    rounding is 0.43 units (RMS over the results' mantissas) and a row takes
    three (two filters and the factor s) besides one of s itself: 0.87; bound
    1.2 (three columns).  A dozen roundings a row give 1.3 to 2.6."""
    import torch
    dev = require_gpu()
    L = np.longdouble
    case = _case((8, 8, nz), (1, 1, 0), seed=3)
    alpha, dt = 0.5, 0.5
    case.params = dict(case.params, c=2.0 * alpha * dt, nu_f=beta / (alpha * dt) * case.h ** 2)
    rng = np.random.default_rng(nz)
    plan = ibmx.Plan.from_case(case, "f64")
    zero = torch.zeros((3, nz, 8, 8), dtype=torch.float64, device=dev)
    for sx, sy in ((1, 1), (-1, 1), (1, -1), (-1, -1)):
        d = rng.normal(size=(3, nz))
        sign = (float(sy) ** np.arange(8))[:, None] * float(sx) ** np.arange(8)
        u = torch.as_tensor(d[:, :, None, None] * sign, device=dev).contiguous()
        plan.fluid_helmholtz(u, zero, zero[0], dt)
        plan.check("helmholtz")
        got = u.cpu().numpy()[:, :, 0, 0]
        b1 = L(alpha) * L(dt) * L(case.params["nu_f"]) / L(case.h) ** 2
        lam = L(-4 * (sx < 0) - 4 * (sy < 0))
        # (1 - b1 (lam - 2)) x_k - b1 (x_k-1 + x_k+1) = d_k, ghosts -x at the walls
        cp, y, prev, last = [], d.astype(L), L(0), L(0)
        for k in range(nz):
            diag = 1 - b1 * (lam - 2 - (k == 0) - (k == nz - 1))
            den = diag + b1 * prev
            last = y[:, k] = (y[:, k] + b1 * last) / den
            prev = -b1 / den
            cp.append(prev)
        for k in range(nz - 2, -1, -1):
            y[:, k] -= cp[k] * y[:, k + 1]
        e = float(np.sqrt(np.mean((got - y) ** 2) / np.mean(y ** 2))) * 2.0 ** 53
        print(f"{nz} {beta:.4f} {sx:+d} {sy:+d}: {e:.2f}", flush=True)
        assert e <= 1.2
    plan.close()

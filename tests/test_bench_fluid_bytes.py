"""Bytes by which bench.py rates the fluid steps against the memory: what the
kernels move, never more than the textbook forms."""
import os
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_moved_bytes_of_the_solves():
    n, N = (512, 512, 512), 512 ** 3
    # y passes 32 B per node, the solve along z 16
    assert bench.fluid_moved("helmholtz", 4, n) == 3 * (2 * 4 + 8 + 48 + 8 + 4) * N
    rim = 4 * (1 / 64 + 1 / 4 + 1 / 32)
    assert bench.fluid_moved("project", 4, n) == pytest.approx(
        (3 * 4 + 8 + 16 + 48 + 16 + 8 + 11 * 4 + 2 * rim) * N)
    assert bench.fluid_moved("predictor", 8, n) == 16 * 8 * N
    with pytest.raises(KeyError):
        bench.fluid_moved("other", 4, n)


@pytest.mark.parametrize("nz,walls,z", [(15, True, 32), (16, True, 16), (2048, True, 16),
                                        (2049, True, 32), (8, False, 16), (1024, False, 16)])
def test_solve_along_z_by_its_route(nz, walls, z):
    n = (8, 8, nz)
    assert bench.fluid_moved("helmholtz", 8, n, walls) == 3 * (16 + 8 + 32 + z + 8 + 8) * 64 * nz


@pytest.mark.parametrize("kind", ["predictor", "helmholtz", "project"])
@pytest.mark.parametrize("walls", [0, 1])
def test_fraction_of_peak_by_moved_bytes(kind, walls):
    case = types.SimpleNamespace(n=(512, 512, 512), periodic=(1, 1, 1 - walls))
    r = bench.fluid_roofline(kind, case, 10.0)
    moved = bench.fluid_moved(kind, 4, case.n, bool(walls))
    assert r["bytes"] == moved <= bench.fluid_bytes(kind, 4, 512 ** 3, bool(walls))
    assert r["frac"] == pytest.approx(moved / 1e-2 / 8e12, abs=1e-4)
    assert r["textbook_GBs"] >= r["achieved_GBs"]

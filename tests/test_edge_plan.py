"""How the fused edge kernels divide the atoms (host code of tests/device/probe.hip; CPU only)."""
import ctypes

import pytest

from paper_2506_04055_amd.build import probe_lib


@pytest.fixture(scope="module")
def atoms():
    f = ctypes.CDLL(probe_lib()).probe_atoms_per_workgroup
    f.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_float, ctypes.c_float, ctypes.c_int]
    return lambda n, degree, slots=60: f(n, int(n * degree * 1.1 ** 3), 5.0, 0.5, slots)


@pytest.mark.parametrize("degree", [0.1, 0.5, 1, 2, 4, 8, 12, 16, 20, 31, 52, 100, 150, 400])
def test_a_run_fills_its_rows(atoms, degree):
    n = 200_000
    a = atoms(n, degree)
    run = min(60, a, max(1, int(128 // degree)))          # atoms of one run
    # at least half of the rows, unless the slots or a single atom set the limit
    assert run * degree >= 64 or run in (1, 60)
    assert a <= 64


@pytest.mark.parametrize("n", [1, 5, 192, 1000, 1536, 3000, 10_000, 16_000])
@pytest.mark.parametrize("degree", [0.0, 0.5, 4, 16, 52, 150])
def test_small_systems_use_every_compute_unit(atoms, n, degree):
    a = atoms(n, degree)
    assert 1 <= a <= max(6, -(-n // 256))


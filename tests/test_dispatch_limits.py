"""Sizes at which a launch rule has to leave a form whose indices would not
hold them (rules of the host code: no GPU)."""
import ctypes

import pytest


class Dims(ctypes.Structure):
    _fields_ = [("nx", ctypes.c_int), ("ny", ctypes.c_int), ("nz", ctypes.c_int)]


@pytest.fixture(scope="module")
def nslib():
    from paper_2206_07732_amd import ns
    ns.lib()
    return ns


# (the marched level set takes two pseudo-steps per launch, the one-cell form one)
@pytest.mark.parametrize("grid,steps", [((512, 256, 256), 2), ((23170, 23169, 2), 2), ((23171, 23171, 2), 1),
                                        ((4, 134217729, 2), 1)])
def test_marched_level_set_keeps_its_planes_in_32_bit_offsets(nslib, grid, steps):
    P = nslib.NSParams()
    P.nx, P.ny, P.nz = grid
    P.h = P.rho_w = P.rho_a = P.rho_s = P.mu_w = P.mu_a = P.mu_s = P.n_cells = 1.0
    assert nslib.lib().ns_workspace_bytes(ctypes.byref(P)) > 0, "a valid grid"
    assert (8 * max((grid[0] + 1) * grid[1], grid[0] * (grid[1] + 1)) < 2 ** 32) == (steps == 2)
    rule = ctypes.CDLL(nslib.LIB_PATH)._ZN3nsk12reinit_stepsERKNS_4DimsE
    assert rule(ctypes.byref(Dims(*grid))) == steps

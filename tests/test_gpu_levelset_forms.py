"""The level-set stage on each side of the rules that pick its form (advection
marched or not; pseudo-steps marched two or one to a launch, or by a cell per
lane) against the oracle: flat and narrow grids, ragged tiles of the forms with
two steps and with one, odd counts of steps that end on a single one; and with
infinities and a NaN in the level set, whose cells and neighbourhoods the marched
forms must leave as the one-cell form does."""
import ctypes

import numpy as np
import pytest

from gates import Scales, gate
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# grid, pseudo-steps, steps per launch
CASES = [((200, 72, 104), 5, 2), ((187, 113, 81), 5, 2), ((16, 257, 260), 3, 2), ((124, 125, 97), 5, 2),   # two
         ((64, 509, 65), 5, 1), ((513, 16, 301), 2, 1), ((127, 64, 300), 3, 1),                            # one, marched
         ((512, 4, 513), 3, 1), ((1024, 4, 259), 2, 1), ((64, 128, 129), 4, 1)]                            # one-cell


def _steps(grid):
    from paper_2206_07732_amd import ns
    ns.lib()
    rule = ctypes.CDLL(ns.LIB_PATH)._ZN3nsk12reinit_stepsERKNS_4DimsE
    return rule((ctypes.c_int * 3)(*grid))


def _case(grid):
    nx, ny, nz = grid
    wl = I.workload("c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    rng = np.random.default_rng(6)
    for k in ("u", "v", "w"):   # a face speed of about 0.3 everywhere, the walls' zero
        f[k] += rng.uniform(-0.3, 0.3, f[k].shape)
    f["u"][:, :, [0, -1]] = 0.0
    f["v"][:, [0, -1], :] = 0.0
    f["w"][0] = 0.0
    f["sigma"] += rng.uniform(-0.5, 0.5, f["sigma"].shape) * wl.h
    return wl, f, 0.2 * wl.h


def _run(wl, f, dt, iters):
    from paper_2206_07732_amd import ns
    dev = ns.device_fields(f)
    S = ns.Solver(ns.params(wl, reinit_iters=iters), dev)
    S.levelset_advect_reinit(dt)
    torch.cuda.synchronize()
    S.close()
    return dev["sigma"].cpu().numpy()


@pytest.mark.parametrize("grid,iters,per", CASES, ids=lambda g: "x".join(map(str, g)) if isinstance(g, tuple) else str(g))
def test_stage_parity(orc, grid, iters, per):
    assert np.prod(grid) >= 1 << 20 and _steps(grid) == per
    wl, f, dt = _case(grid)
    P = orc.params(wl, reinit_iters=iters)
    ref = orc.reinit(P, orc.levelset_advect(P, f["sigma"], f["u"], f["v"], f["w"], dt))
    gate(f"{grid} sigma", _run(wl, f, dt, iters), ref, 1e-13, Scales(wl, f, dt).L)


@pytest.mark.parametrize("grid,low,iters", [((187, 113, 81), 48, 5), ((64, 509, 65), 32, 3)],
                         ids=lambda g: "x".join(map(str, g)) if isinstance(g, tuple) else str(g))
def test_values_that_are_not_finite(grid, low, iters):
    """The lower planes of the same tank by themselves take the one-cell forms."""
    nx, ny, nz = grid
    assert nx * ny * nz >= 3 << 19 and nx * ny * low < 1 << 20
    wl, f, dt = _case(grid)
    for v, (k, j, i) in zip((np.inf, -np.inf, np.nan, np.inf, -np.inf),
                            ((20, 30, 40), (9, 14, 62), (25, 70, 61), (0, 0, 0), (15, ny - 1, nx - 1))):
        f["sigma"][k, j, i] = v
    whole = _run(wl, f, dt, iters)
    wl2, f2, _ = _case((nx, ny, low))
    wl2.h = wl.h
    for k in ("sigma", "u", "v"):
        f2[k] = np.ascontiguousarray(f[k][:low])
    f2["w"] = np.ascontiguousarray(f["w"][:low + 1])
    part = _run(wl2, f2, dt, iters)
    m = low - iters - 3   # (what the planes above reach)
    a, b = whole[:m], part[:m]
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.isnan(a).any()
    assert np.array_equal(np.isposinf(a), np.isposinf(b)) and np.array_equal(np.isneginf(a), np.isneginf(b))
    fin = np.isfinite(b)
    assert fin.sum() > 0.9 * fin.size
    assert np.max(np.abs(a[fin] - b[fin])) <= 1e-13 * nz * wl.h

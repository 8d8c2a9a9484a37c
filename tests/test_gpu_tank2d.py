"""The 2-D levels' one-launch visits (a tile of 64 x 8 cells and a ring of
four) against the oracle at the sizes where they can go wrong: one tile in
part, tiles cut by the far walls by two cells or one row, a tank one cell pair
past a tile, levels whose next one is another 2-D launch, the tail's, or a
coarsest level too large for the tail; and the sweep counts they do not take."""
import numpy as np
import pytest

from gates import Scales, gate, gate_fields, host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(256, 1, 64),    # 2 levels of launches, then the tail
         (66, 1, 42),     # 33 x 21 below, the tail's
         (130, 1, 18),    # one cell pair and two rows past the tiles
         (192, 1, 8),     # one tile high
         (380, 1, 188),   # 95 x 47 coarsest
         (254, 1, 138)]   # 127 x 69 coarsest: too large for the tail


def _case(grid):
    nx, ny, nz = grid
    wl = I.workload("c1", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    return wl, I.make_fields(wl)


def _solver(wl, f, **opts):
    from paper_2206_07732_amd import ns
    dev = ns.device_fields(f)
    return ns.Solver(ns.params(wl, **opts), dev), dev


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 5e-7)])
def test_vcycle_parity(orc, grid, prec, tol):
    wl, f = _case(grid)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    for nu in (2, 1):
        S, _ = _solver(wl, f, prec=prec, nu_pre=nu)
        S.momentum_step(dt, dt)
        x = np.random.default_rng(3).standard_normal(f["p"].shape)
        zo = orc.vcycle(orc.params(wl, prec=prec, nu_pre=nu), *(host(S.buffer(k)) for k in ("bx", "by", "bz")), x)
        z = torch.empty(x.shape, dtype=torch.float64, device="cuda")
        S.vcycle(torch.from_numpy(x).cuda(), z)
        torch.cuda.synchronize()
        gate(f"{grid} V-cycle prec={prec} nu={nu}", z, zo, tol, float(np.max(np.abs(zo))))
        S.close()


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_step_parity_and_replay(orc, grid):
    """A step with the CG count forced against the oracle's, and replayed graphs
    bit for bit what single launches leave, in both precisions."""
    from paper_2206_07732_amd import ns
    wl, f = _case(grid)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    opts = dict(max_iters=5, rtol=0.0)
    ref, _, _ = orc.step(orc.params(wl, **opts), f, dt, 0.0)
    for prec in (0, 1):
        outs = []
        for mode in (ns.LAUNCH_GRAPH, ns.LAUNCH_STREAM):
            S, dev = _solver(wl, f, prec=prec, **opts)
            S.set_launch_mode(mode)
            S.step(dt, 0.0, allow_noconv=True)
            torch.cuda.synchronize()
            if prec == 0 and mode == ns.LAUNCH_GRAPH:
                gate_fields(f"{grid} step", dev, ref, ("sigma", "u", "v", "w", "p"), 1e-10, Scales(wl, f, dt))
            S.step(dt, dt, allow_noconv=True)
            torch.cuda.synchronize()
            outs.append(dev)
            S.close()
        for k in outs[0]:
            assert torch.equal(outs[0][k], outs[1][k]), (prec, k)

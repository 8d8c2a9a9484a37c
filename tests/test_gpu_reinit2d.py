"""A 2-D tank's reinitialisation (up to five pseudo-steps per launch, tiles of
64 x 16 cells) against the oracle: tanks of less than a tile, one cell past a
tile both ways, and counts of pseudo-steps on each side of one and two launches."""
import numpy as np
import pytest

from gates import Scales, gate
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("iters", [1, 4, 5, 6, 11])
@pytest.mark.parametrize("grid", [(4, 5), (64, 16), (65, 17), (131, 50)], ids=lambda g: "x".join(map(str, g)))
def test_stage_parity(orc, grid, iters):
    from paper_2206_07732_amd import ns
    nx, nz = grid
    wl = I.workload("c1", nx=nx, ny=1, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    rng = np.random.default_rng(6)
    f["sigma"] += rng.uniform(-0.5, 0.5, f["sigma"].shape) * wl.h
    dt = 0.1 * wl.h
    P = orc.params(wl, reinit_iters=iters)
    ref = orc.reinit(P, orc.levelset_advect(P, f["sigma"], f["u"], f["v"], f["w"], dt))
    dev = ns.device_fields(f)
    S = ns.Solver(ns.params(wl, reinit_iters=iters), dev)
    S.levelset_advect_reinit(dt)
    torch.cuda.synchronize()
    gate(f"{grid} sigma, {iters} steps", dev["sigma"], ref, 1e-13, Scales(wl, f, dt).L)
    S.close()

"""The level-set stage in the form larger grids take (columns marched in z,
two pseudo-steps per launch) against the oracle at the sizes where it can go
wrong: rows of one tile in part, one lane past a tile, planes of one chunk in
part, heights of a few planes, every count of pseudo-steps' parity, and a state
with velocities through the open top."""
import numpy as np
import pytest

from gates import Scales, gate
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid,iters", [((128, 128, 64), 5), ((127, 131, 65), 2), ((63, 130, 129), 1), ((1025, 257, 4), 4),
                                        ((62, 30, 566), 3), ((311, 4, 845), 0)],
                         ids=lambda g: "x".join(map(str, g)) if isinstance(g, tuple) else str(g))
def test_stage_parity(orc, grid, iters):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    assert nx * ny * nz >= 1 << 20
    wl = I.workload("c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    rng = np.random.default_rng(6)
    for k in ("u", "v", "w"):   # a face speed of about 0.3 everywhere, the walls' zero
        f[k] += rng.uniform(-0.3, 0.3, f[k].shape)
    f["u"][:, :, [0, -1]] = 0.0
    f["v"][:, [0, -1], :] = 0.0
    f["w"][0] = 0.0
    f["sigma"] += rng.uniform(-0.5, 0.5, f["sigma"].shape) * wl.h
    dt = 0.2 * wl.h
    P = orc.params(wl, reinit_iters=iters)
    ref = orc.reinit(P, orc.levelset_advect(P, f["sigma"], f["u"], f["v"], f["w"], dt))
    dev = ns.device_fields(f)
    S = ns.Solver(ns.params(wl, reinit_iters=iters), dev)
    S.levelset_advect_reinit(dt)
    torch.cuda.synchronize()
    gate(f"{grid} sigma", dev["sigma"], ref, 1e-13, Scales(wl, f, dt).L)
    S.close()

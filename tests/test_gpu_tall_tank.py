"""The predictor's one-launch form on tanks whose planes, taken three times, pass
the 65536 blocks a launch may have along z: against the oracle."""
import numpy as np
import pytest

from gates import Scales, gate, gate_velocity
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [(2, 2, 40000), (2, 1, 90000), (3, 2, 30000)], ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("consistent", [0, 1])
def test_predictor(orc, grid, consistent):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    h = 2.0 / nz
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=h, bodies=[], consistent=consistent)
    f = I.make_fields(wl)
    rng = np.random.default_rng(4)
    for k in ("u", "v", "w"):
        f[k] += rng.uniform(-0.1, 0.1, f[k].shape)
    f["u"][:, :, [0, -1]] = 0.0
    f["v"][:, [0, -1], :] = 0.0
    f["w"][0] = 0.0
    dt = 0.2 * h
    P = orc.params(wl)
    S = ns.Solver(ns.params(wl), ns.device_fields(f))
    S.momentum_step(dt, dt)
    torch.cuda.synchronize()
    if consistent:
        ref, rb = orc.momentum_cons(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt, orc.properties(P, f["sigma"], 0.0)[0])
        beta = orc.face_beta_rho(P, rb, f["sigma"], dt, dt)
    else:
        ref = orc.momentum(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt)
        beta = orc.face_beta(P, f["sigma"], dt, dt)
    sc = Scales(wl, f, dt)
    gate_velocity(f"predictor {grid}", [S.buffer(k) for k in ("us", "vs", "ws")], ref, ("us", "vs", "ws"), 1e-13, sc)
    for k, r in zip(("bx", "by", "bz"), beta):
        gate(f"beta {grid} {k}", S.buffer(k), r, 1e-13, sc.of(k, r))
    S.close()

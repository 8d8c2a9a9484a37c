"""The predictor and its Crank-Nicolson sweeps in the form larger grids take
(two faces along x per lane) against the oracle at the sizes where it can go
wrong: rows of an odd length, of two and three cells, one pair past a
wavefront; a 2-D tank; bodies, the inlet and the damping zone of a wave tank."""
import dataclasses

import numpy as np
import pytest

from gates import Scales, gate, gate_velocity
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = {"even": (130, 44, 37), "odd": (127, 49, 33), "two": (2, 331, 300), "three": (3, 257, 256), "tank2d": (1025, 1, 193)}


def _case(name, tank=False, **over):
    nx, ny, nz = GRIDS[name]
    h = 2.0 / nz
    assert nx * ny * nz >= 3 << 16
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=h, **over)
    if tank:
        wl = dataclasses.replace(wl, nwt={"gen": 0.2 * nx * h, "damp": 0.3 * nx * h, "vort": 4 * h})
    f = I.make_fields(wl)
    rng = np.random.default_rng(4)
    for k in ("u", "v", "w"):
        f[k] += rng.uniform(-0.1, 0.1, f[k].shape)
    f["u"][:, :, [0, -1]] = 0.0
    f["v"][:, [0, -1], :] = 0.0
    f["w"][0] = 0.0
    f["sigma"] += rng.uniform(-0.5, 0.5, f["sigma"].shape) * h
    return wl, f, 0.2 * h


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("consistent", [0, 1])
def test_predictor_parity(orc, name, consistent):
    from paper_2206_07732_amd import ns
    wl, f, dt = _case(name, tank=name in ("odd", "tank2d"), consistent=consistent)
    P = orc.params(wl)
    S = ns.Solver(ns.params(wl), ns.device_fields(f))
    S.momentum_step(dt, dt)
    torch.cuda.synchronize()
    if consistent:
        rho_n = orc.properties(P, f["sigma"], 0.0)[0]
        ref, rb = orc.momentum_cons(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt, rho_n)
        beta = orc.face_beta_rho(P, rb, f["sigma"], dt, dt)
    else:
        ref = orc.momentum(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt)
        beta = orc.face_beta(P, f["sigma"], dt, dt)
    sc = Scales(wl, f, dt)
    gate_velocity(f"predictor {name}", [S.buffer(k) for k in ("us", "vs", "ws")], ref, ("us", "vs", "ws"), 1e-13, sc)
    for k, r in zip(("bx", "by", "bz"), beta):
        gate(f"beta {name} {k}", S.buffer(k), r, 1e-13, sc.of(k, r))
    S.close()


@pytest.mark.parametrize("name", list(GRIDS))
def test_sweeps_solve_the_same_system_as_one_face_per_lane(orc, name):
    """u* of the Crank-Nicolson predictor satisfies D u* - L(u*)/2 = rhs: one
    more batch of sweeps from it moves no face by more than the tolerance that
    ended the first (a face left out, or written from a wrong neighbour, would
    keep the sweeps from converging)."""
    from paper_2206_07732_amd import ns
    wl, f, dt = _case(name)
    out = []
    for tol, sweeps in ((1e-14, 2), (1e-14, 7)):
        S = ns.Solver(ns.params(wl, cn_sweeps=sweeps, cn_tol=tol), ns.device_fields(f))
        S.momentum_step(dt, dt)
        torch.cuda.synchronize()
        out.append([S.buffer(k).clone() for k in ("us", "vs", "ws")])
        S.close()
    top = max(float(a.abs().max()) for a in out[0])
    for a, b in zip(*out):
        assert float((a - b).abs().max()) <= 1e-13 * top

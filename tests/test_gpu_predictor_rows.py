"""The predictor of larger grids at the row lengths where its form changes (one
face along x per lane below 64 cells, two from there on), and the Crank-Nicolson
sweeps of both forms, against the oracle: odd rows, whose last pair is half
one, rows of two and three cells, 2-D tanks, a wave tank's inlet and damping
zone, both forms of the transport."""
import dataclasses

import numpy as np
import pytest

from gates import Scales, gate, gate_velocity, host, velocity_norm
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = {"two": (2, 331, 300), "three": (3, 257, 256), "short": (63, 57, 56), "short2d": (33, 1, 5959),   # one face
         "row64": (64, 56, 56), "row65": (65, 56, 55), "even": (130, 44, 37), "odd": (127, 49, 33),       # two
         "tank2d": (1025, 1, 193)}


def _case(name, tank, **over):
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


def _oracle(orc, wl, f, dt):
    P = orc.params(wl)
    if wl.consistent:
        return orc.momentum_cons(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt, orc.properties(P, f["sigma"], 0.0)[0])
    return orc.momentum(P, f["u"], f["v"], f["w"], f["sigma"], dt, dt), None


@pytest.mark.parametrize("name", ["short", "short2d", "row64", "row65"])
@pytest.mark.parametrize("consistent", [0, 1])
def test_predictor(orc, name, consistent):
    from paper_2206_07732_amd import ns
    wl, f, dt = _case(name, True, consistent=consistent)
    P = orc.params(wl)
    S = ns.Solver(ns.params(wl), ns.device_fields(f))
    S.momentum_step(dt, dt)
    torch.cuda.synchronize()
    ref, rb = _oracle(orc, wl, f, dt)
    beta = orc.face_beta_rho(P, rb, f["sigma"], dt, dt) if consistent else orc.face_beta(P, f["sigma"], dt, dt)
    sc = Scales(wl, f, dt)
    gate_velocity(f"predictor {name}", [S.buffer(k) for k in ("us", "vs", "ws")], ref, ("us", "vs", "ws"), 1e-13, sc)
    for k, r in zip(("bx", "by", "bz"), beta):
        gate(f"beta {name} {k}", S.buffer(k), r, 1e-13, sc.of(k, r))
    S.close()


# one viscosity for both phases, nu dt / h^2 = 0.02 in the lighter one: the sweeps
# contract by some ten there and faster elsewhere (a face of air beside water's
# viscosity is past the sweeps' bound), the term moves the velocity by percents,
# and 1e-14 of the last sweep's change leaves the system solved to 1e-12
@pytest.mark.parametrize("name,tank,consistent", [(n, n in ("short", "row65"), 0) for n in GRIDS] +
                         [("short", False, 1), ("odd", False, 1)])
def test_crank_nicolson(orc, name, tank, consistent):
    from paper_2206_07732_amd import ns
    h = 2.0 / GRIDS[name][2]
    mu = 0.02 * h / 0.2 * I.workload("c3").rho_a
    over = dict(mu_w=mu, mu_a=mu, mu_s=mu, consistent=consistent)
    wl, f, dt = _case(name, tank, cn_sweeps=3, **over)
    S = ns.Solver(ns.params(wl, cn_tol=1e-14), ns.device_fields(f))
    S.momentum_step(dt, dt)
    torch.cuda.synchronize()
    got = [host(S.buffer(k)).copy() for k in ("us", "vs", "ws")]
    S.close()
    ref = _oracle(orc, wl, f, dt)[0]
    assert orc.last_flags() == 0
    gate_velocity(f"Crank-Nicolson {name}", got, ref, ("us", "vs", "ws"), 1e-12, Scales(wl, f, dt))
    ex = _oracle(orc, _case(name, tank, cn_sweeps=0, **over)[0], f, dt)[0]
    assert velocity_norm([r - e for r, e in zip(ref, ex)]) > 1e-4 * velocity_norm(ref), "the term is well above the gate"

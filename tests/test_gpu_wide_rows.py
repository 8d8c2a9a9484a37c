"""The finest level's passes with several cell pairs per lane and the
colour-split CG vectors, which large levels with long rows take, against the
oracle at the sizes where they can go wrong: rows that fill a wavefront in
part (48, 49 or 101 lanes of two pairs, 48 of four in FP32), rows and planes
that do not fill a tile, odd extents, and a single level, whose solve keeps
its vectors in natural order."""
import numpy as np
import pytest

from gates import Scales, gate, gate_fields, host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = {"w384": (384, 56, 52), "w404": (404, 66, 42), "w196": (196, 75, 73)}


def _case(name):
    nx, ny, nz = GRIDS[name]
    h = 2.0 / nz
    wl = I.workload("c3", nx=nx, ny=ny, nz=nz, h=h, bodies=[I.Body(1, (0.4 * nx * h, 0.5 * ny * h, 0.0), (0.25, 0.7, 1.5))])
    return wl, I.make_fields(wl)


def _solver(wl, f, **opts):
    from paper_2206_07732_amd import ns
    dev = ns.device_fields(f)
    return ns.Solver(ns.params(wl, **opts), dev), dev


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 5e-7)])
def test_vcycle_parity(orc, name, prec, tol):
    wl, f = _case(name)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    S, _ = _solver(wl, f, prec=prec)
    S.momentum_step(dt, dt)
    x = np.random.default_rng(8).standard_normal(f["p"].shape)
    zo = orc.vcycle(orc.params(wl, prec=prec), *(host(S.buffer(k)) for k in ("bx", "by", "bz")), x)
    for tables in (False, True):
        S.set_face_tables(tables)
        z = torch.empty(x.shape, dtype=torch.float64, device="cuda")
        S.vcycle(torch.from_numpy(x).cuda(), z)
        torch.cuda.synchronize()
        gate(f"{name} V-cycle prec={prec} tables={tables}", z, zo, tol, float(np.max(np.abs(zo))))
    S.close()


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("nu", [1, 2])
def test_step_parity_forced_iterations(orc, name, nu):
    wl, f = _case(name)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    opts = dict(max_iters=6, rtol=0.0, nu_pre=nu, nu_post=nu)
    ref, _, _ = orc.step(orc.params(wl, **opts), f, dt, 0.0)
    outs = []
    for tables in (False, True):
        S, dev = _solver(wl, f, **opts)
        S.set_face_tables(tables)
        assert S.step(dt, 0.0, allow_noconv=True)["iters"] == 6
        torch.cuda.synchronize()
        outs.append(dev)
        S.close()
    gate_fields(f"{name} step", outs[0], ref, ("sigma", "u", "v", "w", "p"), 1e-10, Scales(wl, f, dt))
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("name", ["w384", "w404"])
def test_converged_steps_mixed_and_replayed(orc, name):
    """The FP32 cycle reaches the FP64 cycle's state, and replayed graphs leave
    bit for bit what single launches leave."""
    from paper_2206_07732_amd import ns
    wl, f = _case(name)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    out = {}
    for prec, mode in ((0, ns.LAUNCH_GRAPH), (1, ns.LAUNCH_GRAPH), (1, ns.LAUNCH_STREAM)):
        S, dev = _solver(wl, f, prec=prec)
        S.set_launch_mode(mode)
        for s in range(3):
            assert S.step(dt, s * dt)["true_rel_resid"] <= 1e-10
        torch.cuda.synchronize()
        out[prec, mode] = dev
        S.close()
    a, b, c = out.values()
    gate_fields(f"{name} mixed", b, {k: host(v) for k, v in a.items()}, ("u", "w", "p"), 1e-8, Scales(wl, f, dt))
    for k in b:
        assert torch.equal(b[k], c[k]), k

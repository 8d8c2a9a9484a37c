"""The CG scalars where the updates' kernels sum the partials themselves (up to
512 of them) and one step past that, against the oracle with the CG count
forced; replayed graphs against single launches, and a restart from the true
residual (a first direction in the middle of a solve)."""
import numpy as np
import pytest

from gates import Scales, gate_fields
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(16, 1, 4), (1024, 1, 128), (1028, 1, 128), (64, 64, 32), (68, 64, 32), (33, 7, 5)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_step_parity_and_replay(orc, grid):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    dt = orc.cfl_dt(orc.params(wl), f, wl.cfl, wl.dt_max)
    opts = dict(max_iters=5, rtol=0.0)
    ref, _, _ = orc.step(orc.params(wl, **opts), f, dt, 0.0)
    outs = []
    for mode in (ns.LAUNCH_GRAPH, ns.LAUNCH_STREAM):
        dev = ns.device_fields(f)
        S = ns.Solver(ns.params(wl, **opts), dev)
        S.set_launch_mode(mode)
        S.step(dt, 0.0, allow_noconv=True)
        torch.cuda.synchronize()
        if not outs:
            gate_fields(f"{grid} step", dev, ref, ("sigma", "u", "v", "w", "p"), 1e-10, Scales(wl, f, dt))
        for s in range(1, 3):
            S.step(dt, s * dt, allow_noconv=True)
        torch.cuda.synchronize()
        outs.append(dev)
        S.close()
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k
    # a tolerance below what the recursion can confirm makes the solve restart
    dev = ns.device_fields(f)
    S = ns.Solver(ns.params(wl, max_iters=60, rtol=1e-13), dev)
    st = S.step(dt, 0.0, allow_noconv=True)
    assert np.isfinite(st["true_rel_resid"]) and st["true_rel_resid"] < 1e-11
    S.close()

"""An FP32 cycle whose first coarse level takes four pairs per lane, its rows three
quarters of a wavefront: against the oracle, and with the coarse level's line
tables bit for bit what it gives without them."""
import numpy as np
import pytest

from gates import gate, host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_vcycle_four_pairs_on_a_coarse_level(orc):
    from paper_2206_07732_amd import ns
    nx, ny, nz = 768, 104, 108   # 384 x 52 x 54 below: 1078272 cells
    wl = I.workload("c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    S = ns.Solver(ns.params(wl, prec=1), ns.device_fields(f))
    S.momentum_step(1e-3, 1e-3)
    x = np.random.default_rng(3).standard_normal(f["p"].shape)
    faces = [host(S.buffer(k)) for k in ("bx", "by", "bz")]
    out = []
    for on in (True, False):
        S.set_face_tables(on)
        z = torch.empty(x.shape, dtype=torch.float64, device="cuda")
        S.vcycle(torch.from_numpy(x).cuda(), z)
        torch.cuda.synchronize()
        out.append(z)
    S.close()
    assert torch.equal(out[0], out[1])
    zo = orc.vcycle(orc.params(wl, prec=1), *faces, x)
    gate("768x104x108 V-cycle prec=1", out[0], zo, 5e-7, float(np.max(np.abs(zo))))

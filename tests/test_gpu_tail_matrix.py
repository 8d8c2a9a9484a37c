"""The tail's matrix, which a solve's cycles use and a lone ns_vcycle does not: the
first iterate of a solve from zero is the cycle's correction z = M b times a
number, so its direction is z's.  Against the oracle's FP64 cycle (of the
FP32-rounded operands for the mixed one), with the matrix of the finest level,
of a level below the registers' and of the levels of each product form."""
import numpy as np
import pytest

from gates import host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(8, 4, 8), (16, 1, 16),   # 256 cells, the finest level
         (10, 2, 10),              # 200
         (6, 4, 4), (4, 4, 4), (4, 1, 8),   # 96, 64, 32
         (16, 8, 16), (64, 1, 64), (64, 32, 32), (256, 1, 64)]


# (an FP64 correction is a sum of up to 256 terms, rounded to about 2e-16 with the
# matrix' own entries as far off again, and the oracle's is 2e-16 off; the FP32
# one is rounded to 6e-8 at the matrix, its coefficients and each pass above)
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec,tol", [(0, 5e-16), (1, 3e-7)])
def test_first_direction(orc, grid, prec, tol):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    dev = ns.device_fields(f)
    S = ns.Solver(ns.params(wl, prec=prec, max_iters=1, rtol=0.0), dev)
    S.momentum_step(1e-3, 1e-3)
    r32 = (lambda a: a.astype(np.float32).astype(np.float64)) if prec else (lambda a: a)
    faces = [r32(host(S.buffer(k))) for k in ("bx", "by", "bz")]
    rng = np.random.default_rng(6)
    err = 0.0
    for _ in range(4):
        b = r32(rng.standard_normal(f["p"].shape))
        S.buffer("rhs").copy_(torch.from_numpy(b))
        dev["p"].zero_()
        S.pcg_solve(allow_noconv=True)
        torch.cuda.synchronize()
        z = orc.vcycle(orc.params(wl), *faces, b)
        p = host(dev["p"])
        err += float(np.sum((p / np.linalg.norm(p) - z / np.linalg.norm(z)) ** 2)) / 4
    S.close()
    print(f"[tail matrix] {grid} prec={prec}: {err ** 0.5:.2e}", flush=True)
    assert err ** 0.5 <= tol

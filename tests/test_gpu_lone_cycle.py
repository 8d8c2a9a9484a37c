"""A lone ns_vcycle runs every level by passes, without the matrix that a solve
forms for its cycles: on grids and tails that are a matrix in a solve, its FP64
correction is as near the oracle's as two cycles of passes are."""
import numpy as np
import pytest

from gates import host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (each cycle is some 2e-16 from the exact one; a product of 256 terms summed one
# after the other is 5e-16 off by itself)
@pytest.mark.parametrize("grid", [(8, 4, 8), (16, 1, 16), (8, 8, 4), (2, 2, 2), (4, 1, 2), (6, 4, 4), (16, 8, 16), (24, 18, 14)],
                         ids=lambda g: "x".join(map(str, g)))
def test_passes_throughout(orc, grid):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    S = ns.Solver(ns.params(wl), ns.device_fields(f))
    S.momentum_step(1e-3, 1e-3)
    faces = [host(S.buffer(k)) for k in ("bx", "by", "bz")]
    rng = np.random.default_rng(6)
    err = 0.0
    for _ in range(4):
        b = rng.standard_normal(f["p"].shape)
        z = torch.empty(b.shape, dtype=torch.float64, device="cuda")
        S.vcycle(torch.from_numpy(b).cuda(), z)
        torch.cuda.synchronize()
        want = orc.vcycle(orc.params(wl), *faces, b)
        err += float(np.sum((host(z) - want) ** 2) / np.sum(want ** 2)) / 4
    S.close()
    print(f"[lone cycle] {grid}: {err ** 0.5:.2e}", flush=True)
    assert err ** 0.5 <= 4e-16

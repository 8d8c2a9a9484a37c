"""ns_vcycle with z on r: in place, and with the two arrays overlapping in part,
bit for bit what separate arrays give; 2-D levels of many tiles, whose visits
read r to the end, and every other form of a cycle's first and last kernel."""
import numpy as np
import pytest

from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(256, 1, 64), (640, 1, 96), (1024, 1, 256), (66, 1, 42), (16, 1, 16), (24, 18, 14), (128, 64, 64), (192, 84, 66)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec", [0, 1])
def test_overlapping_arrays_give_the_separate_ones_result(grid, prec):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    S = ns.Solver(ns.params(wl, prec=prec), ns.device_fields(f))
    S.momentum_step(1e-3, 1e-3)
    n = nx * ny * nz
    x = torch.from_numpy(np.random.default_rng(3).standard_normal(n)).cuda()
    want = torch.empty_like(x)
    S.vcycle(x, want)
    for off in (0, nx, -3 * nx - 1):   # z's first entry after r's
        buf = torch.zeros(n + abs(off), dtype=torch.float64, device="cuda")
        r, z = (buf[:n], buf[off:off + n]) if off >= 0 else (buf[-off:-off + n], buf[:n])
        for _ in range(3):
            r.copy_(x)
            S.vcycle(r, z)
            torch.cuda.synchronize()
            assert torch.equal(z, want), (off, float((z - want).abs().max()))
    S.close()

"""A V-cycle's error against extended precision on the levels held in registers
and the 2-D levels' one-launch visits: that of the same cycle in numpy, in the
cycle's precision with every update divided by its diagonal, as the separate
passes divide (a product with the rounded 1/D is 1.5 to 2.8 times as far off)."""
import numpy as np
import pytest

from paper_2206_07732_amd import inputs as I
from test_gpu_wall_faces import _cycle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(25, 9, 13),     # one level of registers
         (49, 9, 13),     # the same in FP32; FP64: separate passes
         (130, 1, 18),    # a 2-D visit; 65 x 9 below, in registers
         (66, 1, 42)]     # the same; 33 x 21 below


# (two cycles that round in another order: their errors, each the root mean
# square of a thousand cells and more and of four right-hand sides, agree to a tenth)
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec", [0, 1])
def test_error_is_that_of_dividing_passes(grid, prec):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    h = 2.0 / nz
    T = np.float32 if prec else np.float64
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=h, bodies=[])
    S = ns.Solver(ns.params(wl, prec=prec), ns.device_fields(I.make_fields(wl)))
    S.momentum_step(1e-3, 1e-3)
    faces = [S.buffer(k).cpu().numpy().astype(T) for k in ("bx", "by", "bz")]
    rng = np.random.default_rng(2)
    err = {"gpu": 0.0, "numpy": 0.0}
    for _ in range(4):
        b = rng.standard_normal((nz, ny, nx)).astype(T)
        ref = _cycle(np.longdouble(h), *(a.astype(np.longdouble) for a in faces), b.astype(np.longdouble))
        z = torch.empty((nz, ny, nx), dtype=torch.float64, device="cuda")
        S.vcycle(torch.from_numpy(b.astype(np.float64)).cuda(), z)
        for k, v in (("gpu", z.cpu().numpy()), ("numpy", _cycle(T(h), *faces, b))):
            err[k] += float(np.sum((v - ref) ** 2) / np.sum(ref ** 2)) / 4
    S.close()
    e = {k: v ** 0.5 for k, v in err.items()}
    print(f"[cycle accuracy] {grid} prec={prec}: {e['gpu']:.2e}, numpy {e['numpy']:.2e}", flush=True)
    assert e["gpu"] <= 1.2 * e["numpy"]

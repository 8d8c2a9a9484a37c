"""Coefficients written through ns_buffer with nonzero walls: the levels held in
registers and the 2-D levels' one-launch visits drop a wall's neighbour term, as
the separate passes do, instead of reading the entry that lies beyond it.  The
reference is a V-cycle in numpy: red-black Gauss-Seidel with a cell's six
faces in its diagonal and no term through a wall."""
import numpy as np
import pytest

from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [(25, 9, 13),     # one level of registers, 1521 pairs
         (63, 1, 65),     # the same, 2-D
         (49, 9, 13),     # FP32: registers, 2925 pairs; FP64: separate passes
         (254, 1, 138)]   # a 2-D visit; 127 x 69 below, separate passes


def _neighbour_sum(n, h, bx, by, bz, e):
    """sum of beta e_nb over the faces that are no walls (the top has none)"""
    s = np.zeros_like(e)
    s[:, :, 1:] += bx[:, :, 1:-1] * e[:, :, :-1]
    s[:, :, :-1] += bx[:, :, 1:-1] * e[:, :, 1:]
    s[:, 1:] += by[:, 1:-1] * e[:, :-1]
    s[:, :-1] += by[:, 1:-1] * e[:, 1:]
    s[1:] += bz[1:-1] * e[:-1]
    s[:-1] += bz[1:-1] * e[1:]
    return s


def _residual(n, h, bx, by, bz, b, e):
    a = np.zeros_like(e)
    d = bx[:, :, 1:-1] * (e[:, :, 1:] - e[:, :, :-1])
    a[:, :, 1:] += d
    a[:, :, :-1] -= d
    d = by[:, 1:-1] * (e[:, 1:] - e[:, :-1])
    a[:, 1:] += d
    a[:, :-1] -= d
    d = bz[1:-1] * (e[1:] - e[:-1])
    a[1:] += d
    a[:-1] -= d
    a[-1] += 2.0 * bz[-1] * e[-1]
    return b - a / h ** 2


def _cycle(h, bx, by, bz, b, nu=2, sweeps=10):
    n = b.shape
    k, j, i = np.indices(n)
    colour = (i + j + k) & 1
    diag = bx[:, :, :-1] + bx[:, :, 1:] + by[:, :-1] + by[:, 1:] + bz[:-1] + bz[1:]
    diag[-1] += bz[-1]
    e = np.zeros_like(b)

    def passes(first, count):
        for s in range(count):
            v = (h * h * b + _neighbour_sum(n, h, bx, by, bz, e)) / diag
            e[colour == (first + s) % 2] = v[colour == (first + s) % 2]

    if any(m % 2 for m in n if m > 1):
        passes(0, 2 * sweeps)
        passes(1, 2 * sweeps)
        return e
    assert n[1] == 1   # (a 2-D tank: x and z are halved)
    passes(0, 2 * nu)
    half = lambda a: 0.25 * (a[::2, :, ::2] + a[1::2, :, ::2] + a[::2, :, 1::2] + a[1::2, :, 1::2])
    cbx, cbz = 0.5 * (bx[::2, :, ::2] + bx[1::2, :, ::2]), 0.5 * (bz[::2, :, ::2] + bz[::2, :, 1::2])
    ec = _cycle(2 * h, cbx, half(by), cbz, half(_residual(n, h, bx, by, bz, b, e)))
    e += np.repeat(np.repeat(ec, 2, axis=0), 2, axis=2)
    passes(1, 2 * nu)
    return e


# (FP32: some 44 passes of a dozen roundings of 6e-8 each, half of them up)
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-5)])
def test_wall_faces_that_are_not_zero(grid, prec, tol):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    h = 2.0 / nz
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=h, bodies=[])
    S = ns.Solver(ns.params(wl, prec=prec), ns.device_fields(I.make_fields(wl)))
    S.momentum_step(1e-3, 1e-3)
    rng = np.random.default_rng(8)
    faces = []
    for k in ("bx", "by", "bz"):
        buf = S.buffer(k)
        faces.append(rng.uniform(0.5, 1.0, size=tuple(buf.shape)).astype(np.float32).astype(np.float64))
        buf.copy_(torch.from_numpy(faces[-1]))
    b = rng.standard_normal((nz, ny, nx))
    want = _cycle(h, *faces, b)
    z = torch.empty((nz, ny, nx), dtype=torch.float64, device="cuda")
    S.vcycle(torch.from_numpy(b).cuda(), z)
    torch.cuda.synchronize()
    err = float(np.max(np.abs(z.cpu().numpy() - want)) / np.max(np.abs(want)))
    print(f"[wall faces] {grid} prec={prec}: {err:.2e}", flush=True)
    assert err <= tol
    S.close()

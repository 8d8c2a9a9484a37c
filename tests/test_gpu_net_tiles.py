"""The inference network's forward in the tile forms it chooses by the grid, at
the sizes where they can go wrong, against the oracle's bfloat16 emulation
(tolerance as in test_gpu_net.py): two rows and 16 channels per block, four
rows, eight rows; tiles cut by every far wall; averages fused into a cut tile.
Larger grids are compared on windows at two opposite corners and inside: values
16 cells or more from a window's artificial edge do not depend on what lies
beyond it (the layers reach 1 + 2 + 4 + 2 + 1 cells, and the averages round
that up to their cells)."""
import numpy as np
import pytest

from gates import gate
from oracle import net_oracle as N

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MARGIN, W = 16, 40


def _windows(dims):
    """Per window and axis: the cells [lo, hi) taken, and those judged."""
    def axis(n, at):
        lo = {"lo": 0, "mid": max(0, (n - W) // 8 * 4), "hi": max(0, n - W)}[at]
        hi = min(n, lo + W)
        return lo, hi, lo if lo == 0 else lo + MARGIN, hi if hi == n else hi - MARGIN
    return [[axis(n, at) for n in dims] for at in ("lo", "mid", "hi")]


@pytest.mark.parametrize("dims", [(4, 4, 4), (36, 20, 12), (68, 36, 36), (100, 68, 52), (164, 76, 100)],
                         ids=lambda d: "x".join(map(str, d)))
def test_forward_tiles(dims):
    from paper_2206_07732_amd import ns
    nx, ny, nz = dims
    rng = np.random.default_rng(sum(dims))
    theta = N.he_init(5)
    theta[-161:] = rng.standard_normal(161) * 0.05
    feat = rng.standard_normal((4, nz, ny, nx)).astype(np.float32)
    net = ns.Net(nx, ny, nz)
    net.set_params(theta)
    f = torch.from_numpy(feat).cuda()
    out = net.forward(f).cpu().numpy()
    assert np.array_equal(out, net.forward(f).cpu().numpy())
    net.close()
    th = N.unflatten(theta.astype(np.float32).astype(np.float64))
    for x, y, z in _windows(dims):
        win = feat[:, z[0]:z[1], y[0]:y[1], x[0]:x[1]]
        ref, _ = N.forward(th, win.astype(np.float64), bf16=True)
        r = ref[z[2] - z[0]:z[3] - z[0], y[2] - y[0]:y[3] - y[0], x[2] - x[0]:x[3] - x[0]]
        o = out[z[2]:z[3], y[2]:y[3], x[2]:x[3]]
        gate(f"net forward {dims} at {x[2], y[2], z[2]}", o, r, 5e-3, float(np.max(np.abs(ref))))

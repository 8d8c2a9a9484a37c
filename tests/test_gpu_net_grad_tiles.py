"""The network's gradients on grids whose levels fill the weight gradient's
16 x 4 x 2 tiles in part, in every direction, against the oracle's BF16
emulation.  Features, weights and biases are positive, so every
pre-activation is far from the ReLU's kink: what differs between the two
sides is the summation order, which now and then flips a BF16 rounding (2^-9
of one value), and with signed weights such a flip can also open or close a
ReLU and move whole gradients by a per cent on a small grid.  Tolerance 5e-3,
as for the other gradient tests."""
import numpy as np
import pytest

from gates import gate
from oracle import net_oracle as N
from test_gpu_net import random_beta

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dims", [(4, 4, 4), (20, 12, 8), (36, 20, 12), (68, 8, 4)])
def test_gradients_on_partial_tiles(orc, dims):
    from paper_2206_07732_amd import ns
    nx, ny, nz = dims
    rng = np.random.default_rng(sum(dims))
    theta = np.abs(N.he_init(11)) * 0.2
    theta[-161:] = np.abs(rng.standard_normal(161)) * 0.05
    feat = (0.5 + rng.random((4, nz, ny, nx))).astype(np.float32)
    target = (rng.standard_normal((nz, ny, nx)) * 0.3).astype(np.float32)
    b, beta = random_beta(nx, ny, nz, 4)
    net = ns.Net(nx, ny, nz, training=True)
    net.set_params(theta)
    loss = net.train_step(torch.from_numpy(feat).cuda(), torch.from_numpy(target).cuda(), beta, 1e-3, update=False)
    G = N.unflatten(net.get_grads().astype(np.float64))
    out, cache = N.forward(N.unflatten(theta.astype(np.float32).astype(np.float64)), feat.astype(np.float64), bf16=True)
    op = lambda x: orc.apply_A(nx, ny, nz, 1.0, *(a.astype(np.float64) for a in b), x)  # noqa: E731
    L, dout = N.energy_loss_and_grad(out, target.astype(np.float64), op)
    assert abs(loss - L) < 5e-3 * L
    for k, ref in N.backward(cache, dout).items():
        gate(f"net grad {dims} {k}", G[k], ref, 5e-3, float(np.max(np.abs(ref))))

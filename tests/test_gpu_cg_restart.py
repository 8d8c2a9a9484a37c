"""A solve that restarts from its true residual.  A guess a thousand million times
the solution leaves rounding in the recursion's residual far above the
tolerance, so its first confirmation must fail and the solve go on with a first
direction in its middle: with the CG scalars folded into the updates' kernels (up
to 512 partials), with finalizing launches, and with colour-split vectors."""
import numpy as np
import pytest

from gates import host
from paper_2206_07732_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

RTOL = 1e-9


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", [(16, 1, 16), (256, 1, 64), (64, 64, 32), (68, 64, 32), (192, 84, 66)],
                         ids=lambda g: "x".join(map(str, g)))
def test_restart(orc, grid, prec):
    from paper_2206_07732_amd import ns
    nx, ny, nz = grid
    wl = I.workload("c1" if ny == 1 else "c3", nx=nx, ny=ny, nz=nz, h=2.0 / nz, bodies=[])
    f = I.make_fields(wl)
    rng = np.random.default_rng(9)
    b = torch.from_numpy(rng.standard_normal(f["p"].shape)).cuda()

    def solve(max_iters, guess, mode=ns.LAUNCH_GRAPH):
        dev = ns.device_fields(f)
        S = ns.Solver(ns.params(wl, prec=prec, rtol=RTOL, max_iters=max_iters), dev)
        S.set_launch_mode(mode)
        S.momentum_step(1e-3, 1e-3)
        S.buffer("rhs").copy_(b)
        dev["p"].copy_(guess)
        st = S.pcg_solve(allow_noconv=True)
        torch.cuda.synchronize()
        A = [host(S.buffer(k)) for k in ("bx", "by", "bz")]
        S.close()
        return st, dev["p"].clone(), A

    zero = torch.zeros_like(b)
    st0, want, A = solve(200, zero)
    assert st0["status"] == ns.NS_OK
    guess = 1e9 * float(want.abs().max()) * torch.from_numpy(rng.standard_normal(f["p"].shape)).cuda()
    st, p, _ = solve(200, guess)
    assert st["status"] == ns.NS_OK and st["true_rel_resid"] <= RTOL
    # stopped at the iteration of a failed confirmation, a solve reports that
    # true residual as its last one; stopped at another past the first, the recursion's
    failed = [k for k in range(2, st["iters"])
              if (s := solve(k, guess)[0])["rel_resid"] == s["true_rel_resid"] > RTOL]
    print(f"[restart] {grid} prec={prec}: failed confirmations at {failed} of {st['iters']} iterations", flush=True)
    assert failed
    st2, q, _ = solve(200, guess, ns.LAUNCH_STREAM)
    assert st2["iters"] == st["iters"] and torch.equal(p, q)
    # both solve A p = b to 1e-9 of ||b||: their difference has a residual of 2e-9
    d = host(p) - host(want)
    r = orc.apply_A(nx, ny, nz, wl.h, *A, d)
    assert np.linalg.norm(r) <= 3.0 * RTOL * float(b.norm())

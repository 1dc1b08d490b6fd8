"""The advection-diffusion passes at the edges of their tiles (64 and 128 columns, halo rows,
remainders, odd rows, few planes) against the oracle, <= 1e-12 at a fixed number of cycles; the
input is NaN in dead cells, which are never read into a fluid cell."""
import numpy as np
import pytest

from oracle import OracleProblem
from oracle.momentum import MomentumOracle, srj_rho, srj_schedule
from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [(2, 3, 2), (9, 6, 1), (63, 7, 5), (64, 6, 6), (65, 13, 9), (66, 12, 8), (120, 14, 7), (127, 15, 5), (128, 16, 4),
         (129, 29, 12), (131, 31, 13), (30, 40, 50)]


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "x".join(map(str, d)))
def test_momentum_tiles(dims, first):
    import torch

    from paper_2505_17287_amd import ibm

    rng = np.random.default_rng(sum(dims))
    f = [np.concatenate([[0.0], np.cumsum(rng.uniform(0.9, 1.1, n))]) for n in dims]
    c = [0.5 * a[-1] for a in f]
    if dims[2] == 1:
        v, t = I.prism_mesh(0.22 * min(f[0][-1], f[1][-1]), 16, -1.0, 2.0, center=(c[0], c[1]))
    else:
        v, t = I.icosphere(2)
        v = v * 0.34 * min(a[-1] for a in f) + np.array(c)
    P = OracleProblem(*f)
    P.set_mesh(v, t)
    P.classify()
    P.build_stencils()
    mo = MomentumOracle(P)
    g = ibm.Grid(*f)
    g.setup(v, t)
    shape = (3, dims[2], dims[1], dims[0])
    U0, H0 = rng.uniform(-1.0, 1.0, shape), rng.uniform(-1.0, 1.0, shape)
    if dims[2] == 1:
        U0[2] = H0[2] = 0.0
    nu, dt = 0.3, 0.2
    om = srj_schedule(srj_rho(mo.m, 0.5 * nu * dt), 3)
    Ur, Hr, _, _ = mo.step(U0, H0, nu, dt, first=first, omegas=om, fixed_cycles=2)
    dead = P.types() == 2
    Ud = torch.from_numpy(np.where(dead, np.nan, U0)).cuda()
    Hd = torch.from_numpy(H0).cuda()
    code, _ = g.momentum_step(Ud, Hd, nu, dt, first_step=first, m=3, omega=om, fixed_cycles=2)
    scale = max(1.0, np.abs(Ur[:, ~dead]).max())
    assert code == 0
    assert np.max(np.abs(Ud.cpu().numpy() - Ur)[:, ~dead]) <= 1e-12 * scale
    assert np.max(np.abs(Hd.cpu().numpy() - Hr)) <= 1e-12 * max(1.0, np.abs(Hr).max())
    assert not Ud.cpu().numpy()[:, dead].any()

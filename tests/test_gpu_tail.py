"""The one-workgroup tail of the V-cycle over the ways it deals out a level's cells: one wave, x
pairs (one or two per thread, odd rows too), the linear order, a tail of a single level."""
import numpy as np
import pytest

from oracle import OracleProblem
from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu

# fine grid -> levels of the tail (a uniform grid halves every axis)
SIZES = {
    "pairs, two a thread": (32, 32, 32),         # 16^3, 8^3, 4^3, 2^3
    "pairs, odd rows": (30, 30, 34),             # 15 x 15 x 17
    "linear order": (126, 130, 1),               # 63 x 65: 2080 pairs
    "pairs, one a thread": (20, 18, 22),         # 10 x 9 x 11
    "2D square": (128, 128, 1),                  # 64^2
    "long rows": (512, 6, 6),                    # 256 x 3 x 3
    "short rows": (6, 40, 40),                   # 3 x 20 x 20
    "one level": (6, 6, 6),                      # 3^3
}


@pytest.mark.parametrize("name", sorted(SIZES))
@pytest.mark.parametrize("nu", [(2, 2), (0, 1), (1, 0)])
def test_tail_forms(name, nu):
    import torch

    from paper_2505_17287_amd import ibm

    nx, ny, nz = SIZES[name]
    h = 1.0 / 16.0
    f = [I.uniform_faces(0.0, n * h, n) for n in (nx, ny)] + [I.uniform_faces(-0.5 * h, 0.5 * h, 1) if nz == 1
                                                              else I.uniform_faces(0.0, nz * h, nz)]
    if nz == 1:
        v, t = I.prism_mesh(2.2 * h, 64, -1.0, 1.0, center=(0.43 * nx * h, 0.52 * ny * h))
    else:
        v, t = I.icosphere(3)
        v = v * 1.3 * h + np.array([0.43 * nx, 0.52 * ny, 0.47 * nz]) * h
    P = OracleProblem(*f)
    P.set_mesh(v, t)
    P.classify()
    P.build_stencils()
    rhs = np.random.default_rng(5).uniform(-1.0, 1.0, (nz, ny, nx))
    kw = dict(fixed_cycles=2, method="bicgstab", nu1=nu[0], nu2=nu[1])
    ref, _ = P.solve(rhs, **kw)
    active = P.types() != 2
    for precision, tol in (("fp64", 1e-9), ("mixed", 1e-4)):  # mixed: two steps of an FP32 preconditioner
        g = ibm.Grid(*f, precision=precision)
        g.setup(v, t)
        p, _ = g.poisson_solve(torch.from_numpy(rhs).cuda(), precision=precision, **kw)
        err = np.max(np.abs(p.cpu().numpy() - ref)[active]) / np.max(np.abs(ref[active]))
        print(name, nu, precision, "levels", g.levels()[1:], "err", err, flush=True)
        assert err <= tol

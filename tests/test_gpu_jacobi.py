"""The relaxed Jacobi sweep of the scheduled-Jacobi preconditioner on either side of the size at
which its kernel changes, odd and even rows, few planes: one BiCGStab step as the oracle's."""
import numpy as np
import pytest

from oracle import OracleProblem
from oracle.momentum import srj_schedule
from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = {
    "odd rows": lambda: I.wing(45, 24, 31),
    "short rows": lambda: I.wing(6, 30, 30),
    "one plane": lambda: I.cylinder2d(66),
    "one plane, odd rows": lambda: I.cylinder2d(67),
    "past the cache": lambda: I.multibody(224, n_bodies=1, level=3),  # 11.2M cells, 270 MB of fields
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_srj_step(name):
    import torch

    from paper_2505_17287_amd import ibm

    wl = CASES[name]()
    P = OracleProblem.from_workload(wl)
    g, _ = ibm.grid_from_workload(wl)
    rhs = np.random.default_rng(9).uniform(-1.0, 1.0, g.shape)
    m = 3
    om = srj_schedule(max(0.0, np.cos(np.pi / m)), m)
    ref, _ = P.solve(rhs, fixed_cycles=1, method="bicgstab_srj", srj_omega=om)
    p, _ = g.poisson_solve(torch.from_numpy(rhs).cuda(), fixed_cycles=1, method="bicgstab_srj", srj_sweeps=m)
    active = P.types() != 2
    assert np.max(np.abs(p.cpu().numpy() - ref)[active]) <= 1e-9 * np.max(np.abs(ref[active]))

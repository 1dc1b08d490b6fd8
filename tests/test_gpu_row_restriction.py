"""The row-wise restrictions (grids some of whose axes are merged in part) at the edges of their
tiles: finer rows of one window, one more, several; windows of planes that hold no coarse plane's
start; unmerged, halved and partly merged axes; one plane.  A BiCGStab step as the oracle's."""
import numpy as np
import pytest

from oracle import OracleProblem
from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu

# cells per axis and, per axis, the width ratio of the last cell to the first (1: uniform)
CASES = [((61, 12, 14), (1, 1, 1)), ((62, 13, 12), (1, 1, 4)), ((63, 18, 15), (3, 1, 1)), ((122, 9, 11), (1, 6, 1)),
         ((123, 16, 13), (9, 9, 1)), ((125, 30, 1), (1, 5, 1)), ((200, 33, 29), (12, 4, 2)), ((26, 24, 190), (2, 1, 9)),
         ((90, 71, 83), (4, 4, 4))]


def _faces(n, ratio):
    w = np.linspace(1.0, ratio, n)
    return np.concatenate([[0.0], np.cumsum(w)])


@pytest.mark.parametrize("dims,ratios", CASES, ids=lambda v: "x".join(map(str, v)))
def test_step(dims, ratios):
    import torch

    from paper_2505_17287_amd import ibm

    f = [_faces(n, r) for n, r in zip(dims, ratios)]
    c = [a[len(a) // 3] for a in f]
    if dims[2] == 1:
        v, t = I.prism_mesh(3.3, 24, -1.0, 2.0, center=(c[0], c[1]))
    else:
        v, t = I.icosphere(2)
        v = v * 3.3 + np.array(c)
    P = OracleProblem(*f)
    P.set_mesh(v, t)
    P.classify()
    P.build_stencils()
    rhs = np.random.default_rng(sum(dims)).uniform(-1.0, 1.0, (dims[2], dims[1], dims[0]))
    kw = dict(fixed_cycles=1, method="bicgstab")
    ref, _ = P.solve(rhs, **kw)
    active = P.types() != 2
    for precision, tol in (("fp64", 1e-9), ("mixed", 1e-4)):  # mixed: an FP32 preconditioner
        g = ibm.Grid(*f, precision=precision)
        g.setup(v, t)
        p, _ = g.poisson_solve(torch.from_numpy(rhs).cuda(), precision=precision, **kw)
        assert np.max(np.abs(p.cpu().numpy() - ref)[active]) <= tol * np.max(np.abs(ref[active])), precision


@pytest.mark.parametrize("dims,ratios", [((61, 47, 1), (3, 1, 1)), ((62, 90, 1), (1, 4, 1)), ((261, 190, 1), (5, 7, 1)),
                                         ((700, 333, 1), (12, 3, 1)), ((150, 130, 2), (6, 4, 1))],
                         ids=lambda v: "x".join(map(str, v)))
def test_grids_of_one_plane(dims, ratios):
    """One plane (levels of one plane too) and, next to it, two."""
    test_step(dims, ratios)

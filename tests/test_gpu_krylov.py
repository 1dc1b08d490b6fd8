"""The vector and ghost-row passes of a BiCGStab step at their edges (an odd cell count, more
ghosts than one round of the ghost-row pass takes, a handful of ghosts, one plane, preconditioners
without a start sweep): two steps as the oracle's."""
import numpy as np
import pytest

from oracle import OracleProblem
from oracle.momentum import srj_schedule
from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _problem(dims, radius):
    from paper_2505_17287_amd import ibm

    f = [np.linspace(0.0, n, n + 1) for n in dims]
    c = np.array([0.5 * n for n in dims])
    if dims[2] == 1:
        v, t = I.prism_mesh(radius, 24, -1.0, 2.0, center=(c[0], c[1]))
    else:
        v, t = I.icosphere(3 if radius < 30 else 5)
        v = v * radius + c
    P = OracleProblem(*f)
    P.set_mesh(v, t)
    P.classify()
    P.build_stencils()
    g = ibm.Grid(*f, precision="mixed")
    g.setup(v, t)
    rhs = np.random.default_rng(sum(dims)).uniform(-1.0, 1.0, (dims[2], dims[1], dims[0]))
    return P, g, rhs


CASES = {
    "odd count": ((35, 33, 31), 7.3, {}),
    "odd plane": ((63, 65, 1), 11.2, {}),
    "few ghosts": ((40, 24, 20), 1.1, {}),
    "many ghosts": ((108, 106, 104), 47.6, {}),  # 41576 of them
    "no pre-smoothing": ((35, 33, 31), 7.3, dict(nu1=0, nu2=2)),
    "jacobi": ((35, 33, 31), 7.3, dict(method="bicgstab_srj")),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_two_steps(name):
    import torch

    dims, radius, kw = CASES[name]
    P, g, rhs = _problem(dims, radius)
    if name == "many ghosts":
        assert np.sum(P.types() == 1) > 32768
    kw = dict(dict(fixed_cycles=2, method="bicgstab"), **kw)
    okw = dict(kw)
    if kw["method"] == "bicgstab_srj":
        okw["srj_omega"] = srj_schedule(np.cos(np.pi / 4), 4)
        kw["srj_sweeps"] = 4
    ref, _ = P.solve(rhs, **okw)
    p, _ = g.poisson_solve(torch.from_numpy(rhs).cuda(), **kw)
    active = P.types() != 2
    # sums of up to 1e6 terms in another order, carried through two steps
    assert np.max(np.abs(p.cpu().numpy() - ref)[active]) <= 1e-9 * np.max(np.abs(ref[active]))


@pytest.mark.parametrize("nu", [(0, 2), (2, 0), (2, 2)])
def test_mixed_start(nu):
    import torch

    P, g, rhs = _problem((35, 33, 31), 7.3)
    r = torch.from_numpy(rhs).cuda()
    kw = dict(method="bicgstab", rel_tol=1e-11, max_cycles=60, nu1=nu[0], nu2=nu[1])
    a, sa = g.poisson_solve(r, precision="fp64", **kw)
    b, sb = g.poisson_solve(r, precision="mixed", **kw)
    assert sa.status == 0 and sb.status == 0
    assert float((a - b).abs().max() / a.abs().max()) <= 1e-8


@pytest.mark.parametrize("kw", [dict(method="bicgstab"), dict(method="bicgstab", precision="mixed"),
                                dict(method="bicgstab_srj", srj_sweeps=4), dict(method="vcycle"),
                                dict(method="bicgstab", nu1=0)], ids=str)
def test_work_ahead_of_the_residual_changes_nothing(kw):
    import torch

    _, g, rhs = _problem((35, 33, 31), 7.3)
    r = torch.from_numpy(rhs).cuda()
    kw = dict(dict(rel_tol=1e-9, max_cycles=40), **kw)
    a, sa = g.poisson_solve(r, **kw)
    g.set_profiling(True)  # the sweeps are timed one by one: nothing is enqueued ahead
    b, sb = g.poisson_solve(r, **kw)
    assert torch.equal(a, b) and (sa.cycles, sa.status) == (sb.cycles, sb.status)


AHEAD = {
    # 1.06e6 cells: the direction alone goes ahead, the step runs the first sweep itself
    "direction": ((104, 102, 100), dict(method="bicgstab")),
    "direction, mixed": ((104, 102, 100), dict(method="bicgstab", precision="mixed")),
    "direction, jacobi": ((104, 102, 100), dict(method="bicgstab_srj", srj_sweeps=4, max_cycles=12)),
    "set steps": ((35, 33, 31), dict(method="bicgstab", fixed_cycles=5)),
    "set cycles": ((35, 33, 31), dict(method="vcycle", fixed_cycles=5)),
    "one step": ((35, 33, 31), dict(method="bicgstab", max_cycles=1)),
    # the shadow residual is restarted between the work ahead and its step
    "restarts": ((35, 33, 31), dict(method="bicgstab_srj", srj_sweeps=2, breakdown_tol=0.3, max_cycles=60)),
    "restarts, mixed": ((35, 33, 31), dict(method="bicgstab", precision="mixed", breakdown_tol=0.9, max_cycles=60)),
    # the recurrence gets below a tolerance that the true residual does not: the solve goes on
    # after the result has been enqueued behind the residual that fails to confirm
    "not confirmed": ((35, 33, 31), dict(method="bicgstab", rel_tol=2e-15)),
}


@pytest.mark.parametrize("name", AHEAD)
def test_work_ahead_is_dropped_or_used_without_a_trace(name):
    import torch

    dims, kw = AHEAD[name]
    _, g, rhs = _problem(dims, 7.3)
    r = torch.from_numpy(rhs).cuda()
    kw = dict(dict(rel_tol=1e-9, max_cycles=40), **kw)
    a, sa = g.poisson_solve(r, **kw)
    g.set_profiling(True)  # nothing is enqueued ahead
    b, sb = g.poisson_solve(r, **kw)
    print(name, sa.cycles, sa.restarts, sa.status, sa.rel_residual)
    assert torch.equal(a, b)
    assert (sa.cycles, sa.status, sa.restarts, sa.rel_residual) == (sb.cycles, sb.status, sb.restarts, sb.rel_residual)
    assert sa.restarts > 0 or "restarts" not in name
    if name == "not confirmed":  # which restarts the recurrences: as many steps without are others
        _, sc = g.poisson_solve(r, **dict(kw, fixed_cycles=sa.cycles))
        assert sa.status == 0 and sa.rel_residual != sc.rel_residual

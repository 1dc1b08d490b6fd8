"""A solve refused for a non-finite right-hand side or guess leaves in p what it started from: the
guess, or zero without one, and zero on dead cells."""
import numpy as np
import pytest

from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", ["rhs", "guess"])
@pytest.mark.parametrize("guess", [False, True])
@pytest.mark.parametrize("kw", [dict(method="vcycle"), dict(method="vcycle", precision="mixed"), dict(method="bicgstab"),
                                dict(method="bicgstab_srj", srj_sweeps=4)], ids=str)
def test_p_keeps_its_start(kw, guess, bad):
    import torch

    from paper_2505_17287_amd import ibm

    if bad == "guess" and not guess:
        pytest.skip("no guess to be bad")
    f = I.uniform_faces(-1.0, 1.0, 22)
    v, t = I.icosphere(2)
    g = ibm.Grid(f, f, f, precision="mixed")
    g.setup(v * 0.55, t)
    dead = g.cell_types() == 2
    gen = torch.Generator(g.device).manual_seed(3)
    rhs, p = (torch.rand(g.shape, dtype=torch.float64, device=g.device, generator=gen) for _ in range(2))
    (rhs if bad == "rhs" else p)[1, 2, 3] = np.nan
    want = torch.where(dead, 0.0, p) if guess else torch.zeros_like(p)
    with pytest.raises(ibm.IBMError, match="non-finite"):
        g.poisson_solve(rhs, p, use_initial_guess=guess, **kw)
    assert torch.equal(p.view(torch.int64), want.view(torch.int64))

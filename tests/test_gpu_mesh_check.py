"""The device's mesh check: what it accepts and refuses, with the host check's messages, and a
handle that keeps its geometry when a mesh is refused."""
import numpy as np
import pytest

from paper_2505_17287_amd import inputs as I

pytestmark = pytest.mark.gpu


def _meshes():
    rng = np.random.default_rng(3)
    v, t = I.icosphere(4)
    v = v * 0.55
    perm = rng.permutation(len(v))
    back = np.argsort(perm)
    tet = np.array([[-0.5, -0.5, -0.5], [0.6, -0.4, -0.4], [-0.4, 0.6, -0.4], [-0.4, -0.4, 0.6]])
    return {
        "tetrahedron": (tet, np.array([[0, 2, 1], [0, 1, 3], [1, 2, 3], [2, 0, 3]], np.int32)),
        "box": I.aabb_mesh((-0.4, -0.5, -0.3), (0.5, 0.4, 0.6)),
        "icosphere": (v, t),
        "renumbered": (v[perm], back[t[rng.permutation(len(t))]].astype(np.int32)),
        "spare vertices": (np.concatenate([v, np.full((700, 3), 0.25)]), t),
    }


def _broken(v, t):
    def edit(f):
        a = t.copy()
        f(a)
        return a

    def flip(a):
        a[-1] = a[-1][::-1]

    def index(x):
        def f(a):
            a[len(a) // 2, 1] = x
        return f

    nan = v.copy()
    nan[t[len(t) // 3, 0], 2] = np.nan
    return [("mesh is not", v, edit(flip)), ("mesh is not", v, t[:-1]),
            ("mesh is not", v, np.concatenate([t, t[:1]])),
            ("degenerate", v, edit(lambda a: a.__setitem__((0, 1), a[0, 0]))),
            ("mesh is not", v, np.concatenate([t, t])), ("out of range", v, edit(index(len(v)))),
            ("out of range", v, edit(index(-1))), ("non-finite", nan, t)]


@pytest.mark.parametrize("name", sorted(_meshes()))
def test_refusals_keep_the_geometry(name):
    import torch

    from paper_2505_17287_amd import ibm

    v, t = _meshes()[name]
    f = I.uniform_faces(-1.0, 1.0, 20)
    g = ibm.Grid(f, f, f)
    g.bind(len(v), 2 * len(t), 8000)
    g.set_geometry(v, t)
    g.classify()
    g.build_ghost_stencils()
    types = g.cell_types()
    rhs = torch.rand(g.shape, dtype=torch.float64, device=g.device, generator=torch.Generator(g.device).manual_seed(1))
    before, _ = g.poisson_solve(rhs)
    for word, bv, bt in _broken(v, t):
        with pytest.raises(ibm.IBMError, match=word):
            g.set_geometry(bv, bt, max_ghosts=8000)
        after, _ = g.poisson_solve(rhs)  # the handle still holds the accepted mesh
        assert torch.equal(after, before), word
    g.classify()
    g.build_ghost_stencils()
    assert torch.equal(g.cell_types(), types)
    again, _ = g.poisson_solve(rhs)
    assert torch.equal(again, before)


def test_refusals_leave_the_solver_memory_alone():
    """A refused mesh is checked in scratch of the set-up: nothing that a solve in flight reads or
    writes changes, the reduction partials (at the end of the workspace) among it."""
    import torch

    from paper_2505_17287_amd import ibm

    v, t = _meshes()["icosphere"]
    f = I.uniform_faces(-1.0, 1.0, 20)
    g = ibm.Grid(f, f, f)
    g.bind(len(v), 2 * len(t), 8000)
    g.set_geometry(v, t)
    g.classify()
    g.build_ghost_stencils()
    g.poisson_solve(torch.rand(g.shape, dtype=torch.float64, device=g.device))
    off = g._ws_ptr - g.ws.data_ptr()
    tail = g.ws[off:off + g.workspace_bytes(*g._caps)][-131072:]
    before = tail.clone()
    for word, bv, bt in _broken(v, t):
        with pytest.raises(ibm.IBMError, match=word):
            g.set_geometry(bv, bt, max_ghosts=8000)
        assert torch.equal(tail, before), word


@pytest.mark.parametrize("name", ["box", "icosphere", "many"])
def test_moves_are_checked_as_new_meshes_are(name):
    """A move takes what set_geometry takes and refuses what it refuses, with the triangles of the
    last mesh (checked on the host if they are few) and with others; the result is a new handle's."""
    from paper_2505_17287_amd import ibm

    v, t = I.icosphere(6) if name == "many" else _meshes()[name]  # 81920: the device's check
    if name == "many":
        v = v * 0.55
    f = I.uniform_faces(-1.0, 1.0, 20)
    g = ibm.Grid(f, f, f)
    g.bind(len(v), 2 * len(t), 8000)
    g.setup(v, t)
    shift = np.array([0.03, -0.02, 0.05])
    for k, tris in enumerate((t, t, t[::-1], t)):
        moved = v + (k + 1) * shift
        for word, bv, bt in _broken(moved, tris):
            if word == "non-finite" or k == 1:
                with pytest.raises(ibm.IBMError, match=word):
                    g.move_geometry(bv, bt)
        g.move_geometry(moved, tris)
        h = ibm.Grid(f, f, f)
        h.setup(moved, tris)
        assert np.array_equal(g.cell_types().cpu().numpy(), h.cell_types().cpu().numpy())
        a, b = g.ghosts(), h.ghosts()
        assert all(np.array_equal(a[q], b[q]) for q in a), (name, k)
        h.close()

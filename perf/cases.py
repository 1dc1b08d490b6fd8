"""Timed cases of the library's public entry points (`paper_2505_17287_amd.ibm.Grid`).

Each case is one call sequence of a program that marches a flow around immersed bodies:
a projection on a resident grid, a projection of a new geometry (classification, stencils
and solve), an advection-diffusion half-step, a whole fractional step, or a move of the
bodies.  Grids, bodies and options are those of the repository's workloads and benchmark,
at other sizes too; fields and body positions come from the seed.

`exact` solves the same discrete equations again in 64 bits with plain torch operations.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2505_17287_amd import ibm
from paper_2505_17287_amd import inputs as I

EXACT_CELLS = 2_300_000  # larger grids: the reference solve would take too long
NU = 1.0e-3              # Re = 1000, as in the benchmark's half-step


def listed():
    return [
        # 2D validation runs (circular cylinder): latency and launch count alone
        dict(name="cylinder2d_128", kind="project", body="cylinder", nx=128, ny=128, nz=1,
             bodies=1, level=0, precision="fp64", method="bicgstab", fixed=0),
        # smallest request of the serving stream: new geometry, mixed precision
        dict(name="request_64_mixed", kind="request", body="multi", nx=64, ny=64, nz=64,
             bodies=2, level=4, precision="mixed", method="bicgstab", fixed=0),
        # an odd-sized grid (no even row, no row of a multiple of 16), stationary V-cycle iteration
        dict(name="project_ragged_vcycle", kind="project", body="multi", nx=97, ny=83, nz=71,
             bodies=2, level=4, precision="fp64", method="vcycle", fixed=0),
        # one step's pressure on a middle-sized grid with stationary bodies
        dict(name="project_128_fp64", kind="project", body="multi", nx=128, ny=128, nz=128,
             bodies=4, level=4, precision="fp64", method="bicgstab", fixed=0),
        # finite wing: strongly stretched, slower convergence, thin body
        dict(name="wing_256x128x128", kind="project", body="wing", nx=256, ny=128, nz=128,
             bodies=1, level=0, precision="fp64", method="bicgstab", fixed=0),
        # whole fractional step (half-step, faces, projection, cell correction) at an uneven size
        dict(name="fractional_144x160x120", kind="fractional", body="multi", nx=144, ny=160, nz=120,
             bodies=4, level=4, precision="fp64", method="bicgstab", fixed=0),
        # the paper's own pressure solver, a set number of outer steps
        dict(name="srj_128", kind="project", body="multi", nx=128, ny=128, nz=128,
             bodies=4, level=4, precision="fp64", method="bicgstab_srj", fixed=6),
        # advection-diffusion half-step of the benchmark grid
        dict(name="momentum_256", kind="momentum", body="multi", nx=256, ny=256, nz=256,
             bodies=8, level=5, precision="fp64", method="bicgstab", fixed=0),
        # every body moved by part of a cell, fresh cells filled
        dict(name="move_256", kind="move", body="multi", nx=256, ny=256, nz=256,
             bodies=8, level=5, precision="fp64", method="bicgstab", fixed=0),
        # the benchmark's step: classification, stencils, solve and correction
        dict(name="request_256_fp64", kind="request", body="multi", nx=256, ny=256, nz=256,
             bodies=8, level=5, precision="fp64", method="bicgstab", fixed=0),
        # a step's pressure in mixed precision on the benchmark grid
        dict(name="project_256_mixed", kind="project", body="multi", nx=256, ny=256, nz=256,
             bodies=8, level=5, precision="mixed", method="bicgstab", fixed=0),
        # one GPU's share of the largest published case
        dict(name="project_384_fp64", kind="project", body="multi", nx=384, ny=384, nz=384,
             bodies=8, level=5, precision="fp64", method="bicgstab", fixed=0),
    ]


def draw(rng):
    kind = rng.choice(["project", "project", "project", "request", "request", "fractional", "momentum", "move"])
    body = "multi"
    if kind == "project":
        body = rng.choice(["multi", "multi", "wing", "cylinder"])
    case = dict(kind=kind, body=body, precision=rng.choice(["fp64", "fp64", "mixed"]),
                method=rng.choice(["bicgstab"] * 5 + ["vcycle"]), fixed=0)
    if body == "cylinder":
        n = int(round(math.exp(rng.uniform(math.log(96), math.log(1024)))))
        case.update(nx=n, ny=n, nz=1, bodies=1, level=0)
        return case
    n = math.exp(rng.uniform(math.log(56), math.log(288)))
    if rng.random() < 0.1 and body == "multi" and kind == "project":  # the paper's solver, middle sizes
        n = math.exp(rng.uniform(math.log(56), math.log(128)))
        case.update(method="bicgstab_srj", precision="fp64", fixed=6)
    if body == "wing":
        case["method"] = "bicgstab"
        n = max(n, 96.0) / math.sqrt(2.0)
        case.update(nx=2 * int(round(n)), ny=int(round(n)), nz=int(round(n)) + rng.randrange(0, 6), bodies=1, level=0)
        return case
    if rng.random() < 0.4:  # the serving stream's cubes
        n = int(round(n / 16.0)) * 16
        dims = [n, n, n]
    else:
        dims = [max(48, int(round(n * math.exp(rng.uniform(-0.2, 0.2))))) for _ in range(3)]
    case.update(nx=dims[0], ny=dims[1], nz=dims[2], bodies=rng.randrange(1, 9), level=rng.choice([4, 4, 5]))
    return case


# ---- inputs --------------------------------------------------------------------------------


@functools.lru_cache(maxsize=32)
def _faces(body, nx, ny, nz):
    if body == "cylinder":
        w = I.cylinder2d(nx)
        return w.xf, w.yf, w.zf
    if body == "wing":
        w = I.wing(nx, ny, nz)
        return w.xf, w.yf, w.zf
    return tuple(I.stretched_faces(-4.0, 4.0, -2.3, 2.3, n) for n in (nx, ny, nz))


@functools.lru_cache(maxsize=16)
def _mesh(body, bodies, level):
    if body == "cylinder":
        return I.prism_mesh(0.5, 256, -1.0, 1.0)
    if body == "wing":
        return I.box_mesh((0.0, 0.0, 0.0), (1.0, 2.0, 0.08), 15.0)
    rng = np.random.default_rng(100 * bodies + level)
    placed = I.place_bodies(rng, bodies, -2.25, 2.25)
    return I.merge_meshes([I.perturbed_sphere(rng, level, R, c) for c, R in placed])


def _body(case, seed):
    """The case's bodies, moved by the seed by up to half a cell per axis."""
    verts, tris = _mesh(case["body"], case["bodies"], case["level"])
    xf, yf, zf = _faces(case["body"], case["nx"], case["ny"], case["nz"])
    h = [np.min(np.diff(f)) for f in (xf, yf, zf)]
    if case["nz"] == 1:
        h[2] = 0.0
    return verts + np.random.default_rng(seed).uniform(-0.5, 0.5, 3) * h, tris


def _smooth(gen, case, device):
    """Three cell fields, each a sum of six low-wavenumber products of cosines, at most 1."""
    shape = (case["nz"], case["ny"], case["nx"])
    out = torch.zeros((3,) + shape, dtype=torch.float64, device=device)
    t = [(torch.arange(n, dtype=torch.float64) + 0.5) / n for n in shape]
    for c in range(3 if case["nz"] > 1 else 2):
        for _ in range(6):
            k = torch.randint(0, 4, (3,), generator=gen)
            ph = 2.0 * math.pi * torch.rand(3, generator=gen, dtype=torch.float64)
            a = torch.randn((), generator=gen, dtype=torch.float64)
            f = [torch.cos(2.0 * math.pi * k[d] * t[d] + ph[d]).to(device) for d in range(3)]
            out[c] += (a.item() * f[0])[:, None, None] * f[1][:, None] * f[2]
        out[c] /= out[c].abs().max()
    return out


def _fields(case, seed, device):
    """Cell velocity of a projection (broadband, uniform in [-1, 1]) or of a half-step (smooth,
    with the previous convective term)."""
    if case["kind"] in ("fractional", "momentum", "move"):
        gen = torch.Generator().manual_seed(seed)
        return _smooth(gen, case, device), _smooth(gen, case, device)
    gen = torch.Generator(device=device).manual_seed(seed)
    shape = (3, case["nz"], case["ny"], case["nx"])
    u = torch.rand(shape, generator=gen, dtype=torch.float64, device=device) * 2.0 - 1.0
    if case["nz"] == 1:
        u[2] = 0.0
    return u, None


def _dt(case):
    """Half the smallest cell width (CFL 1/2 for speeds up to 1)."""
    xf, yf, zf = _faces(case["body"], case["nx"], case["ny"], case["nz"])
    return 0.5 * min(np.min(np.diff(f)) for f in ((xf, yf) if case["nz"] == 1 else (xf, yf, zf)))


def _solver(case):
    return dict(rel_tol=1e-10, precision=case["precision"], method=case["method"], fixed_cycles=case["fixed"])


def prepare(case, seed):
    grid = ibm.Grid(*_faces(case["body"], case["nx"], case["ny"], case["nz"]), precision=case["precision"])
    verts, tris = _body(case, seed)
    grid.setup(verts, tris)
    U, H = _fields(case, seed, grid.device)
    s = dict(case=case, grid=grid, verts=verts, tris=tris, U=U, H=H, dt=_dt(case), turn=0)
    if case["kind"] in ("project", "request", "fractional"):
        s["faces"] = tuple(torch.empty(sh, dtype=torch.float64, device=grid.device) for sh in grid.face_shapes())
        s["p"] = torch.empty(grid.shape, dtype=torch.float64, device=grid.device)
    if case["kind"] in ("fractional", "momentum", "move"):
        s["Un"] = torch.empty_like(U)  # u^n and H^{n-1} are kept by the program (steps may be retried)
        s["Hn"] = torch.empty_like(H)
    if case["kind"] == "move":
        h = [np.min(np.diff(f)) for f in (grid.xf, grid.yf, grid.zf)]
        s["there"] = verts + np.array([0.3, -0.2, 0.1]) * h
    return s


def run(s):
    case, grid, dt = s["case"], s["grid"], s["dt"]
    kind = case["kind"]
    if kind in ("project", "request"):
        if kind == "request":  # a new geometry on a grid whose workspace stays resident
            grid.set_geometry(s["verts"], s["tris"])
            grid.classify()
            grid.build_ghost_stencils()
        faces = grid.cell_to_faces(s["U"], s["faces"])
        p, _ = grid.project(*faces, dt=dt, p=s["p"], **_solver(case))
        return dict(p=p, u=faces[0], v=faces[1], w=faces[2])
    U = s["Un"].copy_(s["U"])
    if kind == "move":  # there and back: every pass meets fresh cells on both moves
        for verts in (s["there"], s["verts"]):
            counts, fresh = grid.move_geometry(verts, s["tris"])
            grid.fill_fresh(U)
        return dict(U=U, types=grid.cell_types(), counts=counts, fresh=fresh)
    H = s["Hn"].copy_(s["H"])
    if kind == "momentum":
        grid.momentum_step(U, H, NU, dt)
        return dict(U=U, H=H)
    faces, p, _, _ = grid.fractional_step(U, H, NU, dt, p=s["p"], **_solver(case))
    return dict(U=U, H=H, p=p, u=faces[0], v=faces[1], w=faces[2])


def work(case):
    """Inputs read once and outputs written once (8 bytes a value), and the operations of one
    application of each operator: what no solver can do without, however fast it converges."""
    n = case["nx"] * case["ny"] * case["nz"]
    kind = case["kind"]
    values = {"project": 3 + 3 + 1, "request": 3 + 3 + 1, "momentum": 6 + 6, "fractional": 6 + 6 + 3 + 1, "move": 3 + 3}[kind]
    flops = {"project": 40, "request": 40, "momentum": 200, "fractional": 260, "move": 10}[kind]
    mesh = 0
    if kind in ("request", "move"):
        verts, tris = _mesh(case["body"], case["bodies"], case["level"])
        mesh = 24 * len(verts) + 12 * len(tris) + n
    return {"bytes": float(8 * values * n + mesh), "flops": float(flops * n)}


# ---- the same equations in plain torch, 64 bits ----------------------------------------------


class _Reference:
    """Cells, ghost rows and operators of one geometry."""

    def __init__(self, faces, verts, tris, device):
        self.dev = device
        self.f = [torch.as_tensor(np.asarray(a), dtype=torch.float64, device=device) for a in faces[::-1]]  # z, y, x
        self.c = [0.5 * (a[1:] + a[:-1]) for a in self.f]
        self.w = [a[1:] - a[:-1] for a in self.f]
        self.shape = tuple(len(a) for a in self.c)
        self.axes = [d for d in range(3) if self.shape[d] > 1]
        self.tri = torch.as_tensor(np.asarray(verts)[np.asarray(tris)], dtype=torch.float64, device=device)
        solid = self._inside()
        near = torch.nn.functional.max_pool3d((~solid)[None, None].float(), 3, 1, 1)[0, 0] > 0
        self.fluid, self.ghost = ~solid, solid & near
        self.types = torch.where(solid, torch.where(near, 1, 2), 0).to(torch.uint8)
        self.vol = self.w[0][:, None, None] * self.w[1][:, None] * self.w[2]
        self.V = torch.where(self.fluid, self.vol, 0.0)
        self.g = self.ghost.flatten().nonzero().flatten()
        self.bi, self.ip = self._intercepts(self.g)

    def centre(self, cell):
        nz, ny, nx = self.shape
        return torch.stack([self.c[2][cell % nx], self.c[1][cell // nx % ny], self.c[0][cell // (nx * ny)]], 1)

    def _inside(self):
        """Parity of the surface crossings above each cell centre."""
        nz, ny, nx = self.shape
        x, y = self.c[2].repeat(ny), self.c[1].repeat_interleave(nx)
        cnt = torch.zeros((ny * nx, nz + 1), dtype=torch.int32, device=self.dev)
        a, b, d = self.tri[:, 0], self.tri[:, 1], self.tri[:, 2]
        for t in torch.arange(len(self.tri), device=self.dev).split(max(1, 40_000_000 // (nx * ny))):
            lo, hi = self.tri[t].amin(1).amin(0), self.tri[t].amax(1).amax(0)
            col = ((x >= lo[0]) & (x <= hi[0]) & (y >= lo[1]) & (y <= hi[1])).nonzero().flatten()
            if not len(col):
                continue
            X, Y = x[col, None], y[col, None]

            def edge(p, q):
                return (q[t, 0] - p[t, 0]) * (Y - p[t, 1]) - (q[t, 1] - p[t, 1]) * (X - p[t, 0])

            e = torch.stack([edge(b, d), edge(d, a), edge(a, b)])
            at, k = ((e > 0).all(0) | (e < 0).all(0)).nonzero(as_tuple=True)
            s = e[:, at, k]
            z = (s[0] * a[t[k], 2] + s[1] * b[t[k], 2] + s[2] * d[t[k], 2]) / s.sum(0)
            cnt.index_put_((col[at], torch.searchsorted(self.c[0], z)), torch.ones_like(at, dtype=torch.int32), accumulate=True)
        return (cnt.cumsum(1)[:, :nz] % 2 == 1).T.contiguous().reshape(self.shape)

    def _closest(self, p):
        """Closest surface point: the plane's foot where it is inside a triangle, else an edge point."""
        best = torch.full((len(p),), math.inf, dtype=torch.float64, device=self.dev)
        out = torch.zeros_like(p)
        for t in self.tri.split(max(1, 6_000_000 // max(1, len(p)))):
            P = p[:, None]
            n = torch.linalg.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0])
            cand = P - n * ((P - t[:, 0]) * n).sum(-1, keepdim=True) / (n * n).sum(-1, keepdim=True)
            ok = torch.ones(cand.shape[:2], dtype=torch.bool, device=self.dev)
            for i in range(3):
                v, u = t[:, i], t[:, (i + 1) % 3]
                ok &= (torch.linalg.cross((u - v).expand_as(cand), cand - v) * n).sum(-1) >= 0
            d2 = torch.where(ok, ((P - cand) ** 2).sum(-1), math.inf)
            for i in range(3):
                v, e = t[:, i], t[:, (i + 1) % 3] - t[:, i]
                q = v + e * (((P - v) * e).sum(-1, keepdim=True) / (e * e).sum(-1, keepdim=True)).clamp(0.0, 1.0)
                dq = ((P - q) ** 2).sum(-1)
                cand = torch.where((dq < d2)[..., None], q, cand)
                d2 = torch.minimum(d2, dq)
            m, k = d2.min(1)
            out = torch.where((m < best)[:, None], cand[torch.arange(len(p), device=self.dev), k], out)
            best = torch.minimum(best, m)
        return out

    def _intercepts(self, cell):
        x = self.centre(cell)
        bi = self._closest(x)
        if self.shape[0] == 1:
            bi[:, 2] = x[:, 2]
        return bi, 2.0 * bi - x

    def _basis(self, pt, lo, hi):
        s = [(pt[:, d] - lo[:, d]) / (hi[:, d] - lo[:, d]) for d in range(len(self.axes))]
        one = torch.ones_like(s[0])
        return [s[0] * s[1] * s[2], s[0] * s[1], s[1] * s[2], s[0] * s[2], s[0], s[1], s[2], one] if len(s) == 3 else [s[0] * s[1], s[0], s[1], one]

    def rows(self, cell, bi, at, own):
        """Members and weights of interpolation at `at`; the cell's own slot in the box holds the
        intercept's value (own = "value"), the normal derivative there ("normal") or itself ("cell")."""
        nz, ny, nx = self.shape
        D = len(self.axes)
        box, lo, hi = [], [], []
        for d in range(D):  # x, y(, z)
            c = self.c[2 - d]
            i = (torch.searchsorted(c, at[:, d].contiguous(), right=True) - 1).clamp(0, len(c) - 2)
            box.append(i)
            lo.append(c[i])
            hi.append(c[i + 1])
        lo, hi = torch.stack(lo, 1), torch.stack(hi, 1)
        member, rows = [], []
        for corner in range(1 << D):
            off = [(corner >> d) & 1 for d in range(D)]
            idx = [box[d] + off[d] for d in range(D)]
            m = idx[0] + nx * (idx[1] + ny * (idx[2] if D == 3 else 0))
            pt = torch.stack([self.c[2 - d][idx[d]] for d in range(D)], 1)
            row = torch.stack(self._basis(pt, lo, hi), 1)
            mine = m == cell
            if own == "value":
                row = torch.where(mine[:, None], torch.stack(self._basis(bi, lo, hi), 1), row)
            elif own == "normal":
                x = self.centre(cell)
                n = (bi - x) / torch.linalg.norm(bi - x, dim=1, keepdim=True)
                q = bi[:, :D].clone().requires_grad_(True)
                jac = [torch.autograd.grad(b.sum(), q, retain_graph=True, allow_unused=True)[0] for b in self._basis(q, lo, hi)[:-1]]
                dn = torch.stack([(j * n[:, :D]).sum(1) for j in jac] + [torch.zeros_like(jac[0][:, 0])], 1)
                row = torch.where(mine[:, None], dn, row)
            member.append(torch.where(mine, -1, m))
            rows.append(row)
        A = torch.stack(rows, 1)
        beta = torch.linalg.solve(A.transpose(1, 2).contiguous(), torch.stack(self._basis(at, lo, hi), 1))
        member = torch.stack(member, 1)
        types = torch.where(member < 0, 1, self.types.flatten()[member.clamp(min=0)])
        if bool(((types == 2).any(1) | (types != 0).all(1)).any()):
            raise NotImplementedError("a box with a dead member or no fluid member")
        mine = member < 0
        return member.clamp(min=0), torch.where(mine, 0.0, beta), torch.where(mine, beta, 0.0).sum(1)

    def shaped(self, v, axis):
        return v.reshape([-1 if d == axis else 1 for d in range(3)])

    def laplace(self, p):
        """Flux Laplacian per volume, no flux through the walls."""
        out = torch.zeros_like(p)
        for d in self.axes:
            n = self.shape[d]
            flux = p.diff(dim=d) / self.shaped(self.c[d].diff(), d)
            w = self.shaped(self.w[d], d)
            out.narrow(d, 0, n - 1).add_(flux / w.narrow(d, 0, n - 1))
            out.narrow(d, 1, n - 1).sub_(flux / w.narrow(d, 1, n - 1))
        return out

    def diagonal(self):
        out = torch.zeros(self.shape, dtype=torch.float64, device=self.dev)
        for d in self.axes:
            n, a = self.shape[d], self.shaped(1.0 / self.c[d].diff(), d)
            w = self.shaped(self.w[d], d)
            out.narrow(d, 0, n - 1).sub_(a / w.narrow(d, 0, n - 1))
            out.narrow(d, 1, n - 1).sub_(a / w.narrow(d, 1, n - 1))
        return out

    def to_faces(self, U):
        out = []
        for comp, d in ((0, 2), (1, 1), (2, 0)):
            n = self.shape[d]
            size = list(self.shape)
            size[d] += 1
            f = torch.zeros(size, dtype=torch.float64, device=self.dev)
            if n > 1:
                f.narrow(d, 1, n - 1).copy_(self._mean(U[comp], d))
            out.append(f)
        return out

    def _mean(self, a, d):
        n, w = self.shape[d], self.shaped(self.w[d], d)
        wa, wb = w.narrow(d, 0, n - 1), w.narrow(d, 1, n - 1)
        return (wb * a.narrow(d, 0, n - 1) + wa * a.narrow(d, 1, n - 1)) / (wa + wb)

    def project(self, faces, dt):
        """Pressure with the implicit ghost rows and zero mean, and the corrected faces."""
        div = sum(f.diff(dim=d) / self.shaped(self.w[d], d) for f, d in zip(faces, (2, 1, 0)))
        f = torch.where(self.fluid, div / dt, 0.0)
        member, beta, _ = self.rows(self.g, self.bi, self.ip, "normal")
        diag, total = self.diagonal(), self.V.sum()

        def apply(x):  # fluid rows scaled by the diagonal and projected to zero mean; ghost rows as they are
            r = torch.where(self.fluid, self.laplace(x), 0.0)
            r = torch.where(self.fluid, (r - (self.V * r).sum() / total) / diag, 0.0)
            flat = x.flatten()
            r.view(-1)[self.g] = flat[self.g] - (beta * flat[member]).sum(1)
            return r

        b = torch.where(self.fluid, (f - (self.V * f).sum() / total) / diag, 0.0)
        p = _bicgstab(apply, b)
        p = torch.where(self.fluid | self.ghost, p - (self.V * p).sum() / total, 0.0)
        out = [p]
        for face, d in zip(faces, (2, 1, 0)):
            n, g = self.shape[d], face.clone()
            if n > 1:
                touch = self.fluid.narrow(d, 0, n - 1) | self.fluid.narrow(d, 1, n - 1)
                g.narrow(d, 1, n - 1).sub_(torch.where(touch, dt * p.diff(dim=d) / self.shaped(self.c[d].diff(), d), 0.0))
            out.append(g)
        return out

    def half_step(self, U, H, dt):
        """Ghost rows of u^n, convection, and the Crank-Nicolson solve (body at rest)."""
        member, beta, _ = self.rows(self.g, self.bi, self.ip, "value")

        def ghosts(u):
            u.view(-1)[self.g] = -(beta * u.flatten()[member]).sum(1)
            return u

        U = [ghosts(torch.where(self.fluid | self.ghost, u, 0.0)) for u in U]
        a, diag = 0.5 * NU * dt, self.diagonal()
        newU, newH = [], []
        for c in range(3):
            conv = torch.zeros_like(U[c])
            for d in self.axes:
                n, w = self.shape[d], self.shaped(self.w[d], d)
                flux = self._mean(U[2 - d], d) * self._mean(U[c], d)
                conv.narrow(d, 0, n - 1).sub_(flux / w.narrow(d, 0, n - 1))
                conv.narrow(d, 1, n - 1).add_(flux / w.narrow(d, 1, n - 1))
            conv = torch.where(self.fluid, conv, 0.0)
            b = torch.where(self.fluid, U[c] + dt * (1.5 * conv - 0.5 * H[c]) + a * self.laplace(U[c]), 0.0)

            def apply(x):
                r = torch.where(self.fluid, (x - a * self.laplace(x)) / (1.0 - a * diag), 0.0)
                flat = x.flatten()
                r.view(-1)[self.g] = flat[self.g] + (beta * flat[member]).sum(1)
                return r

            newU.append(_bicgstab(apply, b / (1.0 - a * diag)))
            newH.append(conv)
        return torch.stack(newU), torch.stack(newH)


def _bicgstab(apply, b, tol=1e-13):
    """Solution of apply(x) = b from zero, restarted from its true residual."""
    x, norm = torch.zeros_like(b), torch.linalg.norm(b).item()
    for _ in range(6):
        r = b - apply(x)
        if norm == 0.0 or torch.linalg.norm(r).item() <= tol * norm:
            break
        rh, p = r.clone(), torch.zeros_like(r)
        v, rho, alpha, omega = torch.zeros_like(r), 1.0, 1.0, 1.0
        for k in range(1500):
            new = (rh * r).sum().item()
            if new == 0.0 or omega == 0.0:
                break
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            v, rho = apply(p), new
            alpha = rho / (rh * v).sum().item()
            s = r - alpha * v
            t = apply(s)
            omega = ((t * s).sum() / (t * t).sum().clamp(min=1e-300)).item()
            x += alpha * p + omega * s
            r = s - omega * t
            if torch.linalg.norm(r).item() <= 0.3 * tol * norm:
                break
    return x


def exact(case, seed):
    if case["nx"] * case["ny"] * case["nz"] > EXACT_CELLS or case["fixed"]:
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    verts, tris = _body(case, seed)
    faces = _faces(case["body"], case["nx"], case["ny"], case["nz"])
    U, H = _fields(case, seed, dev)
    dt = _dt(case)
    try:
        if case["kind"] == "move":
            there = verts + np.array([0.3, -0.2, 0.1]) * [np.min(np.diff(f)) for f in faces]
            old = _Reference(faces, verts, tris, dev)
            for v in (there, verts):
                new = _Reference(faces, v, tris, dev)
                cell = ((old.types != 0) & new.fluid).flatten().nonzero().flatten()
                bi, _ = new._intercepts(cell)
                m, beta, own = new.rows(cell, bi, 2.0 * new.centre(cell) - bi, "cell")
                for c in range(3):
                    flat = U[c].view(-1)
                    flat[cell] = (beta * flat[m]).sum(1) / (2.0 - own)
                old = new
            counts = torch.bincount(old.types.flatten().int(), minlength=3)
            return dict(U=U, types=old.types, counts=counts, fresh=len(cell))
        R = _Reference(faces, verts, tris, dev)
        if case["kind"] in ("project", "request"):
            p, u, v, w = R.project(R.to_faces(U), dt)
            return dict(p=p, u=u, v=v, w=w)
        U, H = R.half_step(U, H, dt)
        if case["kind"] == "momentum":
            return dict(U=U, H=H)
        before = R.to_faces(U)
        p, u, v, w = R.project(before, dt)
        for c, (a, b, d) in enumerate(zip(before, (u, v, w), (2, 1, 0))):
            n, change = R.shape[d], b - a
            U[c] += torch.where(R.fluid, 0.5 * (change.narrow(d, 0, n) + change.narrow(d, 1, n)), 0.0)
        return dict(U=U, H=H, p=p, u=u, v=v, w=w)
    except NotImplementedError:
        return None

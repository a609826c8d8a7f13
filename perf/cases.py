"""The work that users of the library have it do, as cases to be timed.

A case is one call sequence of a program around the implicit pressure step:
operator applications (FP64, FP32, residual form, non-conforming meshes,
consistent integration), the pressure system, the coefficient update of a
fixed-point iteration, whole Krylov solves and a training step of the learned
preconditioner.  Meshes and fields are those of the benchmark and the tests:
the periodic unit cube, the terrain-following channel over a Gaussian ridge,
its refinement over the ridge, and a smoothly deformed ("wavy") cube.

``exact`` evaluates the same weak forms in plain torch, FP64, by its own
formulas (no code of the library).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_00384_amd as hx

DEV = "cuda:0"
F64 = torch.float64
LX, LY, LZ, RIDGE, WIDTH = 40000.0, 10000.0, 20000.0, 400.0, 2000.0
SCALE_H, SOUND, DT, GAMMA, PENALTY = 7300.0, 340.0, 1.0, 1.4, 2.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _case(name, kind, mesh, nx, ny, nz, k, **more):
    return dict(name=name, kind=kind, mesh=mesh, nx=nx, ny=ny, nz=nz, k=k, **more)


def listed():
    return [
        # one operator application on the benchmark's periodic 4^3 cube, Q2: the
        # smallest system anyone solves, where a launch is everything
        _case("apply_cube_k2", "apply", "cube", 4, 4, 4, 2, f32=False),
        # the headline: FP64 matvec on the terrain channel (the benchmark's
        # degree sweep has this mesh), larger than every cache
        _case("apply_terrain_k4", "apply", "terrain", 128, 32, 32, 4, f32=False),
        # its FP32 form, the operator inside the mixed solves and V-cycles
        _case("apply_terrain_k4_f32", "apply", "terrain", 128, 32, 32, 4, f32=True),
        # true residual on curved cells with odd counts at a high degree
        _case("residual_wavy_k6", "residual", "wavy", 17, 13, 19, 6),
        # operator on the channel refined over the ridge (2:1 hanging faces)
        _case("apply_refined_k4", "apply", "refined", 32, 8, 16, 4, f32=False),
        # operator with consistent integration (2k+1 points)
        _case("consistent_k4", "consistent", "terrain", 64, 16, 32, 4),
        # the stage's pressure system S = D - C A^-1 B, once per FGMRES step
        _case("pressure_k4", "pressure", "terrain", 64, 32, 32, 4),
        # the coefficient update of a fixed-point iteration and the residual
        # with the new coefficients
        _case("coefficients_k4", "coefficients", "terrain", 64, 32, 32, 4),
        # whole solve, CG with block Jacobi on the benchmark's small channel
        _case("solve_cg_k4", "cg", "terrain", 32, 8, 16, 4),
        # whole solve, CG with the FP32 multigrid V-cycle (the fastest solve of
        # the benchmark), four levels
        _case("solve_multigrid_k4", "multigrid", "terrain", 64, 32, 32, 4, levels=4),
        # whole solve, FGMRES(30) with the learned preconditioner
        _case("solve_learned_k4", "learned", "terrain", 32, 8, 16, 4),
        # one training step of the network (forward, backward, Adam), the
        # trainer's batch
        _case("train_k4", "train", "cube", 4, 4, 4, 4, batch=2048),
    ]


# largest number of dofs drawn for a kind (a drawn case costs no more than the
# largest listed one)
_MOST = dict(apply=16e6, residual=12e6, consistent=4e6, pressure=8e6, coefficients=8e6, cg=1e6,
             fgmres=1e6, learned=6e5, multigrid=4e6)


def draw(rng):
    """One more case: a kind, a degree, and a size log-uniform from a few
    hundred dofs (multigrid and solves: a few thousand) to the kind's most."""
    kind = rng.choice(["apply", "apply", "apply", "residual", "consistent", "pressure",
                       "coefficients", "cg", "fgmres", "learned", "multigrid", "train"])
    k = rng.choice([1, 2, 3, 4, 4, 5, 6, 7])
    if kind == "train":
        return dict(kind=kind, mesh="cube", nx=4, ny=4, nz=4, k=rng.choice([2, 3, 4, 4, 5]),
                    batch=int(round(math.exp(rng.uniform(math.log(64), math.log(4096))))))
    if kind in ("learned", "multigrid", "consistent"):
        k = rng.choice([2, 3, 4, 4, 5])
    mesh = rng.choice(["terrain", "terrain", "cube", "wavy"])
    if kind == "apply" and rng.random() < 0.25:
        mesh = "refined"
    if kind in ("pressure", "multigrid", "learned"):
        mesh = "terrain"
    lo = 5e3 if kind in ("cg", "fgmres", "learned", "multigrid") else 500.0
    dofs = math.exp(rng.uniform(math.log(lo), math.log(_MOST[kind] if mesh != "refined" else 2e6)))
    cells = max(1.0, dofs / (k + 1) ** 3)
    # an aspect of up to 4 : 1 : 2 (x, y, z) with odd counts among them
    side = (cells / 8.0) ** (1.0 / 3.0)
    dims = [max(1, int(round(side * a * math.exp(rng.uniform(-0.25, 0.25))))) for a in (4.0, 1.0, 2.0)]
    while dims[0] * dims[1] * dims[2] * (k + 1) ** 3 > 1.2 * dofs and dims[0] > 1:
        dims[0] -= 1
    c = dict(kind=kind, mesh=mesh, nx=dims[0], ny=dims[1], nz=dims[2], k=k)
    if mesh == "refined":
        c.update(nx=max(4, dims[0]), nz=max(2, dims[2]))
    if kind == "apply":
        c["f32"] = rng.random() < 0.4
    if kind == "multigrid":
        # divisible by 2 for each level
        c["levels"] = rng.choice([2, 3])
        s = 2 ** (c["levels"] - 1)
        for d in ("nx", "ny", "nz"):
            c[d] = max(s, c[d] // s * s)
    return c


# ---------------------------------------------------------------------------
# meshes and fields
# ---------------------------------------------------------------------------

def _geo_degree(case):
    return {"cube": 1, "wavy": 2}.get(case["mesh"], 4)


def _box(case):
    """(lo, hi, periodic) of the case's mesh."""
    if case["mesh"] in ("cube", "wavy"):
        return (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (True, True, True)
    return (-LX / 2, 0.0, 0.0), (LX / 2, LY, LZ), (True, True, False)


def _map(case, X):
    """Positions [..., 3] of the undeformed box, deformed."""
    x, y, z = X.unbind(-1)
    if case["mesh"] == "cube":
        return X
    if case["mesh"] == "wavy":
        t, e = 2.0 * math.pi, 0.04
        sx, sy, sz = torch.sin(t * x), torch.sin(t * y), torch.sin(t * z)
        return torch.stack([x + e * sy * sz, y + e * sz * sx, z + e * sx * sy], -1)
    return torch.stack([x, y, z + RIDGE * torch.exp(-(x / WIDTH) ** 2) * (1.0 - z / LZ)], -1)


def _cells(case):
    """Origin and size of every cell in the undeformed box, the neighbour
    table (cells numbered x fastest; on the refined channel the coarse cells
    outside the refined region, then its children) and the quarter faces."""
    lo, hi, periodic = _box(case)
    dims = np.array([case["nx"], case["ny"], case["nz"]])
    h = (np.array(hi) - np.array(lo)) / dims

    def grid(n):
        i = np.arange(int(np.prod(n)))
        return np.stack([i % n[0], i // n[0] % n[1], i // (n[0] * n[1])], -1)

    def step(pos, n, f):
        """Grid position across face f, and whether it is inside."""
        q = pos.copy()
        d = f // 2
        q[:, d] += 1 if f & 1 else -1
        out = (q[:, d] < 0) | (q[:, d] >= n[d])
        q[:, d] %= n[d]
        return q, ~out | periodic[d]

    def index(q, n):
        return q[:, 0] + n[0] * (q[:, 1] + n[1] * q[:, 2])

    pos = grid(dims)
    if case["mesh"] != "refined":
        nbr = np.empty((len(pos), 6), dtype=np.int64)
        for f in range(6):
            q, ok = step(pos, dims, f)
            nbr[:, f] = np.where(ok, index(q, dims), -1)
        return lo + pos * h, np.broadcast_to(h, pos.shape), nbr, None
    # the middle half in x and the lower half in z, split into eight
    nx, nz = case["nx"], case["nz"]

    def refined(p):
        return (p[:, 0] >= nx // 4) & (p[:, 0] < 3 * nx // 4) & (p[:, 2] < max(1, nz // 2))

    fpos = grid(2 * dims)
    fsel = refined(fpos // 2)
    csel = ~refined(pos)
    cid = np.full(len(pos), -1, dtype=np.int64)
    cid[csel] = np.arange(csel.sum())
    fid = np.full(len(fpos), -1, dtype=np.int64)
    fid[fsel] = csel.sum() + np.arange(fsel.sum())
    cpos, kpos = pos[csel], fpos[fsel]
    nc = len(cpos)
    nbr = np.empty((nc + len(kpos), 6), dtype=np.int64)
    hang = []
    for f in range(6):
        d = f // 2
        q, ok = step(cpos, dims, f)
        nbr[:nc, f] = np.where(ok, np.where(refined(q), -2, cid[index(q, dims)]), -1)
        q, ok = step(kpos, 2 * dims, f)
        inner = refined(q // 2)
        nbr[nc:, f] = np.where(ok, np.where(inner, fid[index(q, 2 * dims)], -2), -1)
        t1, t2 = [(1, 2), (0, 2), (0, 1)][d]
        sel = ok & ~inner
        hang.append(np.stack([cid[index(q // 2, dims)], np.full(len(q), f ^ 1),
                              nc + np.arange(len(q)), kpos[:, t1] % 2 + 2 * (kpos[:, t2] % 2)], -1)[sel])
    org = np.concatenate([lo + cpos * h, lo + kpos * (h / 2)])
    size = np.concatenate([np.broadcast_to(h, cpos.shape), np.broadcast_to(h / 2, kpos.shape)])
    return org, size, nbr, np.concatenate(hang)


def _mesh(case):
    """Geometry nodes [cells, (g+1)^3, 3] (device), neighbours and quarter faces (host)."""
    org, size, nbr, hang = _cells(case)
    g = _geo_degree(case)
    t = torch.arange(g + 1, dtype=F64, device=DEV) / g
    ref = torch.stack(torch.meshgrid(t, t, t, indexing="ij")[::-1], -1).reshape(-1, 3)
    org, size = (torch.from_numpy(np.array(a)).to(DEV) for a in (org, size))
    return _map(case, org[:, None, :] + ref[None] * size[:, None, :]), nbr, hang


def _smooth(xyz, case, gen, modes=5):
    """A seeded smooth field at the positions xyz [3, n]: cosine modes that
    are periodic where the mesh is, plus a little noise."""
    lo, hi, periodic = _box(case)
    u = torch.zeros_like(xyz[0])
    r = torch.rand(modes, 5, dtype=F64, device=DEV, generator=gen).cpu()
    for m in range(modes):
        kx, ky, kz = (int(5 * float(v)) - 2 for v in r[m, :3])
        ph = 2.0 * math.pi * float(r[m, 3])
        a = [2.0 * math.pi * q * (xyz[d] - lo[d]) / (hi[d] - lo[d]) for d, q in enumerate((kx, ky))]
        w = (2.0 if periodic[2] else 1.0) * math.pi * kz * (xyz[2] - lo[2]) / (hi[2] - lo[2])
        u += (2.0 * float(r[m, 4]) - 1.0) * torch.cos(a[0] + a[1] + ph) * torch.cos(w)
    return u + 0.01 * torch.randn(u.shape, dtype=F64, device=DEV, generator=gen)


def _coefficients(xyz, case, gen):
    """alpha, beta at the dofs: the isothermal background on the channel,
    constants on the cube, each with a seeded variation of a few per cent."""
    r = (0.02 + 0.03 * torch.rand(2, dtype=F64, device=DEV, generator=gen)).cpu()
    lo, hi, _ = _box(case)
    s = [2.0 * math.pi * (xyz[d] - lo[d]) / (hi[d] - lo[d]) for d in range(2)]
    va, vb = 1.0 + float(r[0]) * torch.sin(s[0]), 1.0 + float(r[1]) * torch.cos(s[1])
    if case["mesh"] in ("cube", "wavy"):
        return va, 0.01 * vb
    e = torch.exp(xyz[2] / SCALE_H)
    return e * va, (SOUND * DT) ** 2 * e * vb


def _pressure_fields(xyz, case, gen):
    """rho and h of the isothermal background with a seeded variation."""
    a, b = _coefficients(xyz, case, gen)
    e = torch.exp(xyz[2] / SCALE_H)
    return a / e * torch.exp(-xyz[2] / SCALE_H), b / e / (DT * DT) / (GAMMA - 1.0)


def _generator(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000 * int(seed) + salt)
    return g


def _context(case, seed):
    """A context with mesh and coefficients, as a program keeps it."""
    nodes, nbr, hang = _mesh(case)
    ctx = hx.HelmDG(0)
    ctx.setup_mesh(case["k"], nodes.cpu().numpy(), nbr, _geo_degree(case), hang=hang)
    del nodes
    xyz = ctx.dof_coordinates()
    alpha, beta = _coefficients(xyz, case, _generator(seed, 1))
    ctx.set_coefficients(alpha, beta, PENALTY)
    return ctx, xyz, alpha, beta


def _network(k, seed, out_scale):
    """He-uniform weights, zero biases, the last layer scaled down."""
    n = k + 1
    g = _generator(seed, 7)
    parts = []
    for o, i in ((256, n ** 3 + 6 * n * n + 1), (256, 256), (n ** 3, 256)):
        w = (2.0 * torch.rand(o, i, dtype=F64, device=DEV, generator=g) - 1.0) * math.sqrt(6.0 / i)
        parts += [(w * (out_scale if len(parts) == 4 else 1.0)).float().reshape(-1),
                  torch.zeros(o, dtype=torch.float32, device=DEV)]
    return torch.cat(parts)


def _levels(case, ctx, seed):
    """The multigrid hierarchy below ctx: meshes halved in each direction,
    Chebyshev smoothers on Lanczos estimates."""
    ctxs = [ctx]
    for l in range(1, case["levels"]):
        c = dict(case, nx=case["nx"] >> l, ny=case["ny"] >> l, nz=case["nz"] >> l)
        ctxs.append(_context(c, seed)[0])
    for l, c in enumerate(ctxs):
        lo, hi = c.estimate_eigenvalues(
            torch.randn(c.n_dofs, dtype=F64, device=DEV, generator=_generator(seed, 20 + l)), 20)
        if l + 1 == len(ctxs):
            c.set_chebyshev(12, 0.9 * lo, 1.1 * hi)
            break
        c.set_chebyshev(2, 1.1 * hi / 15.0, 1.1 * hi)
        nx, ny, nz = case["nx"] >> l, case["ny"] >> l, case["nz"] >> l
        f = np.arange(nx * ny * nz)
        fx, fy, fz = f % nx, f // nx % ny, f // (nx * ny)
        c.set_multigrid(ctxs[l + 1], fx // 2 + nx // 2 * (fy // 2 + ny // 2 * (fz // 2)),
                        fx % 2 + 2 * (fy % 2) + 4 * (fz % 2))
    return ctxs


# relative residual of the whole solves: tight enough that their solutions do
# not depend on the iteration at which the test first passes
RTOL = 1e-11


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        ctx = _context(case, seed)[0]
        ctx.set_network(_network(case["k"], seed, 0.1).cpu().numpy())
        n = case["k"] + 1
        g = _generator(seed, 3)
        F = torch.randn(case["batch"], n ** 3 + 6 * n * n + 1, dtype=torch.float32, device=DEV, generator=g)
        T = torch.randn(case["batch"], n ** 3, dtype=torch.float32, device=DEV, generator=g).clamp_(-1, 1)
        return dict(kind=kind, ctx=ctx, F=F, T=T)
    ctx, xyz, alpha, beta = _context(case, seed)
    g = _generator(seed, 2)
    s = dict(kind=kind, ctx=ctx)
    b = _smooth(xyz, case, g)
    if kind == "apply":
        s["x"] = b.float() if case["f32"] else b
        s["y"] = torch.empty_like(s["x"])
    elif kind == "residual":
        s.update(b=b, x=_smooth(xyz, case, g), r=torch.empty_like(b))
    elif kind == "coefficients":
        s.update(b=b, x=_smooth(xyz, case, g), r=torch.empty_like(b), alpha=alpha, beta=beta)
    elif kind == "consistent":
        ctx.set_consistent(alpha, beta)
        s.update(x=b, y=torch.empty_like(b))
    elif kind == "pressure":
        rho, h = _pressure_fields(xyz, case, _generator(seed, 1))
        ctx.set_pressure_system(rho, h, GAMMA, DT, PENALTY)
        s["x"] = b
    else:
        s.update(b=b, x=torch.empty_like(b))
        if kind == "cg":
            s["params"] = hx.default_params(method=0, rtol=RTOL)
        elif kind == "fgmres":
            s["params"] = hx.default_params(method=1, rtol=RTOL)
        elif kind == "learned":
            ctx.set_network(_network(case["k"], seed, 0.02).cpu().numpy())
            s["params"] = hx.default_params(method=1, rtol=RTOL, pc=hx.HX_PC_LEARNED)
        elif kind == "multigrid":
            s["levels"] = _levels(case, ctx, seed)
            s["params"] = hx.default_params(method=0, rtol=RTOL, pc=hx.HX_PC_MULTIGRID_MIXED)
    return s


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "apply":
        return ctx.apply_operator(state["x"], state["y"])
    if kind == "residual":
        return ctx.residual(state["b"], state["x"], state["r"])
    if kind == "coefficients":
        ctx.set_coefficients(state["alpha"], state["beta"], PENALTY)
        return ctx.residual(state["b"], state["x"], state["r"])
    if kind == "consistent":
        return ctx.apply_consistent(state["x"], state["y"])
    if kind == "pressure":
        return ctx.apply_pressure_part(hx.HX_PS_SYSTEM, state["x"])
    if kind == "train":
        return ctx.train_step(state["F"], state["T"], 1e-3, want_grad=True, want_loss=False)[1]
    return ctx.solve(state["b"], state["x"], state["params"])[0]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

# iterations that the solves take to RTOL, for the count of their work
_ITERATIONS = dict(cg=110, fgmres=110, learned=110, multigrid=24)


def work(case):
    k, kind = case["k"], case["kind"]
    n = k + 1
    if kind == "train":
        widths = ((n ** 3 + 6 * n * n + 1, 256), (256, 256), (256, n ** 3))
        par = sum((i + 1) * o for i, o in widths)
        # forward, input gradient (not of the first layer), weight gradient;
        # weights and moments read and written, the gradient written
        return dict(flops=2.0 * case["batch"] * (3 * sum(i * o for i, o in widths) - widths[0][0] * 256),
                    bytes=4.0 * (case["batch"] * (widths[0][0] + n ** 3) + 7 * par))
    cells = case["nx"] * case["ny"] * case["nz"]
    if case["mesh"] == "refined":
        cells += 7 * (3 * case["nx"] // 4 - case["nx"] // 4) * case["ny"] * max(1, case["nz"] // 2)
    nd, geo = n ** 3, 24 * (_geo_degree(case) + 1) ** 3
    # inputs and outputs of an operator: x, y, alpha, beta at the nodes, the
    # geometry nodes of the cells; arithmetic of the sum-factorised form
    op = cells * (nd * (8 if case.get("f32") else 16) + nd * 16 + geo)
    fl = cells * (36 * n ** 4 + 24 * nd + 6 * (34 * n ** 3 + 30 * n * n))
    vec = 8 * cells * nd
    if kind == "apply":
        return dict(bytes=op, flops=fl)
    if kind in ("residual", "coefficients"):
        return dict(bytes=op + vec, flops=fl)
    if kind == "consistent":
        q = 2 * k + 1
        fl = cells * (4 * (2 * n ** 3 * q + 3 * n * n * q * q + 4 * n * q ** 3) + 24 * q ** 3
                      + 6 * (2 * n ** 3 + 16 * n * n * q + 20 * n * q * q))
        return dict(bytes=op, flops=fl)
    if kind == "pressure":
        # p in, S p out, rho and h, the geometry; B, A^-1 (three), C and D
        return dict(bytes=op, flops=cells * (132 * n ** 4 + 120 * nd + 6 * 40 * n ** 3))
    it = _ITERATIONS[kind]
    # per iteration the operator and the fused vector passes: CG reads x, r, p,
    # q and writes x, r, p; FGMRES reads the basis twice (15 vectors on average)
    step = dict(cg=op + 7 * vec, fgmres=op + 34 * vec, learned=op + 34 * vec,
                multigrid=op + 7 * vec + 4 * 8 / 7 * (op - vec))[kind]
    flm = dict(cg=1.5, fgmres=1.5, learned=1.5, multigrid=1.0 + 5 * 8 / 7)[kind]
    return dict(bytes=it * step, flops=it * flm * fl)


# ---------------------------------------------------------------------------
# 64-bit values in plain torch
# ---------------------------------------------------------------------------

def _lagrange(nodes, pts):
    """Values and derivatives [len(pts), len(nodes)] of the Lagrange basis."""
    n = len(nodes)
    V, D = np.ones((len(pts), n)), np.zeros((len(pts), n))
    for i in range(n):
        for j in range(n):
            if j != i:
                V[:, i] *= (pts - nodes[j]) / (nodes[i] - nodes[j])
        for m in range(n):
            if m == i:
                continue
            t = np.full(len(pts), 1.0 / (nodes[i] - nodes[m]))
            for j in range(n):
                if j not in (i, m):
                    t = t * (pts - nodes[j]) / (nodes[i] - nodes[j])
            D[:, i] += t
    return V, D


def _gauss(n):
    x, w = np.polynomial.legendre.leggauss(n)
    return 0.5 * (x + 1.0), 0.5 * w


def _lobatto(n):
    inner = np.sort(np.polynomial.legendre.Legendre.basis(n - 1).deriv().roots().real)
    return 0.5 * (np.concatenate([[-1.0], inner, [1.0]]) + 1.0)


def _tp(u, X, Y, Z):
    """Tensor product of 1-D matrices on the last three axes (z, y, x)."""
    u = torch.matmul(u, X.t())
    u = torch.matmul(Y, u)
    s = u.shape
    return torch.matmul(Z, u.reshape(*s[:-2], s[-2] * s[-1])).reshape(*s[:-3], Z.shape[0], s[-2], s[-1])


class _Exact:
    """The weak forms on the case's mesh with an nq-point rule."""

    def __init__(self, case, nq=None):
        self.n = n = case["k"] + 1
        self.nq = nq = nq or n
        g = _geo_degree(case)
        nodes, nbr, hang = _mesh(case)
        self.nc = nodes.shape[0]
        self.X = nodes.reshape(self.nc, g + 1, g + 1, g + 1, 3).permute(0, 4, 1, 2, 3).contiguous()
        self.gl, self.basis = np.arange(g + 1) / g, _lobatto(n)
        self.nbr, self.hang = nbr, hang
        self.q, self.w = _gauss(nq)
        t = self._tab(self.q)
        self.B = t[0]
        gt = self._geo_tab(self.q)
        self.detw, self.Ji = self._jac(self.X, (gt, gt, gt))
        w = torch.from_numpy(self.w).to(DEV)
        self.detw = self.detw * (w[:, None, None] * w[:, None] * w)
        self.t = t
        # volumes and areas of the penalty always by the (k+1)-point rule
        qp, wp = _gauss(n)
        gp = self._geo_tab(qp)
        wp = torch.from_numpy(wp).to(DEV)
        self.wp, self.qp = wp, qp
        self.vol = (self._jac(self.X, (gp, gp, gp))[0] * (wp[:, None, None] * wp[:, None] * wp)).sum((1, 2, 3))
        self.groups = self._faces()

    def dofs(self):
        """Positions of the nodes [3, n_dofs]."""
        V = torch.from_numpy(_lagrange(self.gl, self.basis)[0]).to(DEV)
        return _tp(self.X, V, V, V).permute(1, 0, 2, 3, 4).reshape(3, -1).contiguous()

    def _tab(self, pts):
        return tuple(torch.from_numpy(a).to(DEV) for a in _lagrange(self.basis, np.asarray(pts)))

    def _geo_tab(self, pts):
        return tuple(torch.from_numpy(a).to(DEV) for a in _lagrange(self.gl, np.asarray(pts)))

    @staticmethod
    def _jac(X, tabs):
        """det J and J^-1 [cells, d (ref), i (phys), z, y, x] at a tensor grid
        of points (tables of the x, y, z directions)."""
        cols = []
        for d in range(3):
            m = [tabs[e][1] if e == d else tabs[e][0] for e in range(3)]
            cols.append(_tp(X, *m))          # dX_i / dxi_d: [cells, i, z, y, x]
        a, b, c = cols
        bc, ca, ab = (torch.cross(p, q, dim=1) for p, q in ((b, c), (c, a), (a, b)))
        det = (a * bc).sum(1)
        return det, torch.stack([bc, ca, ab], 1) / det[:, None, None]

    def _side(self, cells, d, end, pts):
        """Tables and J^-1 of cells at tangential points pts = (first, second)
        of the face at `end` in direction d."""
        coords = [None, None, None]
        tang = [e for e in range(3) if e != d]
        coords[d] = np.array([float(end)])
        coords[tang[0]], coords[tang[1]] = pts
        det, Ji = self._jac(self.X[cells], [self._geo_tab(c) for c in coords])
        return dict(cells=cells, tabs=[self._tab(c) for c in coords], det=det, Ji=Ji)

    def _faces(self):
        """Groups of faces {minus side, plus side (None on the boundary), d,
        ds, n, sigma}."""
        groups = []
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
        ids = np.arange(self.nc)

        def add(minus, plus, d, lead, weights, area_of, sig_cells, outward=1.0):
            """minus / plus: (cells, end, pts); lead: the side that gives ds, n."""
            sides = [None if s is None else self._side(s[0], d, s[1], s[2]) for s in (minus, plus)]
            L = sides[lead]
            N = L["Ji"][:, d] * L["det"][:, None]
            ds = torch.linalg.norm(N, dim=1)
            nrm = outward * N / ds[:, None]
            shape = [1, 1, 1]
            tang = [2 - e for e in range(3) if e != d]       # axes among (z, y, x)
            ww = torch.ones(1, 1, 1, dtype=F64, device=DEV)
            for ax in tang:
                s = list(shape)
                s[ax] = -1
                ww = ww * weights.reshape(s)
            grp = dict(sides=sides, d=d, ds=ds * ww, n=nrm, sigma=None)
            if sig_cells is not None:
                # area by the (k+1)-point rule on the leading side
                c, end, p = area_of
                A = self._side(c, d, end, p)
                an = torch.linalg.norm(A["Ji"][:, d] * A["det"][:, None], dim=1)
                wa = torch.ones(1, 1, 1, dtype=F64, device=DEV)
                for ax in tang:
                    s = [1, 1, 1]
                    s[ax] = -1
                    wa = wa * self.wp.reshape(s)
                area = (an * wa).sum((1, 2, 3))
                v = torch.minimum(self.vol[sig_cells[0]], self.vol[sig_cells[1]])
                grp["sigma"] = (PENALTY * self.n ** 2 * area / v)[:, None, None, None]
            groups.append(grp)

        W = torch.from_numpy(self.w).to(DEV)
        for d in range(3):
            m = ids[self.nbr[:, 2 * d + 1] >= 0]
            p = self.nbr[m, 2 * d + 1]
            if len(m):
                m, p = dev(m), dev(p)
                add((m, 1, (self.q, self.q)), (p, 0, (self.q, self.q)), d, 0, W,
                    (m, 1, (self.qp, self.qp)), (m, p))
            for end in (0, 1):
                c = ids[self.nbr[:, 2 * d + end] == -1]
                if len(c):
                    add((dev(c), end, (self.q, self.q)), None, d, 0, W, None, None, 1.0 if end else -1.0)
        if self.hang is not None:
            for f in range(6):
                for s in range(4):
                    r = self.hang[(self.hang[:, 1] == f) & (self.hang[:, 3] == s)]
                    if not len(r):
                        continue
                    C, F, d = dev(r[:, 0]), dev(r[:, 2]), f // 2
                    half = ((s % 2 + self.q) / 2, (s // 2 + self.q) / 2)
                    coarse, fine = (C, f & 1, half), (F, 1 - (f & 1), (self.q, self.q))
                    lead = 1 if f & 1 else 0       # the coarse cell is the minus side when f is a + face
                    add(*((coarse, fine) if f & 1 else (fine, coarse)), d, lead, W,
                        (F, 1 - (f & 1), (self.qp, self.qp)), (C, F))
        return groups

    # -- interpolation to a side's points and back
    def _at(self, u, s, der=False):
        """u [..., cells, n, n, n] at the side's points; with der the three
        reference derivatives."""
        u = u[s["cells"]]
        V = [t[0] for t in s["tabs"]]
        val = _tp(u, *V)
        if not der:
            return val
        return val, [_tp(u, *[s["tabs"][e][1] if e == d else V[e] for e in range(3)]) for d in range(3)]

    def _back(self, out, s, val, der=None):
        V = [t[0].t() for t in s["tabs"]]
        a = _tp(val, *V) if val is not None else 0
        if der is not None:
            for d in range(3):
                a = a + _tp(der[d], *[s["tabs"][e][1].t() if e == d else V[e] for e in range(3)])
        out.index_add_(0, s["cells"], a)

    def _cube(self, u):
        return u.reshape(self.nc, self.n, self.n, self.n)

    def _grads(self, u):
        B, D = self.t
        return [_tp(u, *[D if e == d else B for e in range(3)]) for d in range(3)]

    def set(self, alpha, beta):
        B = self.B
        self.m = _tp(self._cube(alpha), B, B, B) * self.detw
        self.bw = _tp(self._cube(beta), B, B, B) * self.detw
        for g in self.groups:
            g["beta"] = [None if s is None else self._at(self._cube(beta), s) for s in g["sides"]]
        return self

    def apply(self, x):
        """A x."""
        u = self._cube(x.double())
        B, D = self.t
        g = torch.stack(self._grads(u), 1)                       # [cells, d, ...]
        f = self.bw[:, None] * (self.Ji * g[:, :, None]).sum(1)   # beta w grad u: [cells, i, ...]
        f = (self.Ji * f[:, None]).sum(2)                         # [cells, d, ...]
        y = _tp(self.m * _tp(u, B, B, B), B.t(), B.t(), B.t())
        for d in range(3):
            y += _tp(f[:, d], *[D.t() if e == d else B.t() for e in range(3)])
        del g, f
        for grp in self.groups:
            if grp["sides"][1] is None:
                continue
            v, dn, gn = [], [], []
            for s, be in zip(grp["sides"], grp["beta"]):
                val, der = self._at(u, s, True)
                t = [(s["Ji"][:, d] * grp["n"]).sum(1) * be for d in range(3)]
                v.append(val)
                gn.append(t)
                dn.append(sum(a * b for a, b in zip(t, der)))
            jump = v[0] - v[1]
            pen = grp["sigma"] * 0.5 * (grp["beta"][0] + grp["beta"][1])
            c = grp["ds"] * (-0.5 * (dn[0] + dn[1]) + pen * jump)
            h = -0.5 * grp["ds"] * jump
            for s, t, sg in zip(grp["sides"], gn, (1.0, -1.0)):
                self._back(y, s, sg * c, [h * a for a in t])
        return y.reshape(-1)

    def pressure(self, p, rho, h):
        """S p = D p - C A^-1 B p of the pressure system."""
        u = self._cube(p)
        B, D = self.t
        Bt = B.t()
        pq = _tp(u, B, B, B) * self.detw
        hr = self._cube(h * rho)
        Bi = torch.linalg.inv(B)
        rw = _tp(self._cube(rho), B, B, B) * self.detw
        v = [torch.zeros_like(u) for _ in range(3)]
        for e in range(3):
            for d in range(3):
                v[e] -= _tp(pq * self.Ji[:, d, e], *[D.t() if a == d else Bt for a in range(3)])
        for grp in self.groups:
            s0, s1 = grp["sides"]
            hat = self._at(u, s0) if s1 is None else 0.5 * (self._at(u, s0) + self._at(u, s1))
            for e in range(3):
                f = hat * grp["n"][:, e] * grp["ds"]
                self._back(v[e], s0, f)
                if s1 is not None:
                    self._back(v[e], s1, -f)
        v = [_tp(_tp(DT * a, Bi.t(), Bi.t(), Bi.t()) / rw, Bi, Bi, Bi) for a in v]
        y = _tp(pq / (GAMMA - 1.0), Bt, Bt, Bt)
        hq = _tp(hr, B, B, B) * self.detw
        vq = [_tp(a, B, B, B) * hq for a in v]
        for d in range(3):
            f = sum(self.Ji[:, d, e] * vq[e] for e in range(3))
            y += DT * _tp(f, *[D.t() if a == d else Bt for a in range(3)])
        for grp in self.groups:
            if grp["sides"][1] is None:
                continue
            f = 0.0
            for s in grp["sides"]:
                f = f + 0.5 * self._at(hr, s) * sum(self._at(v[e], s) * grp["n"][:, e] for e in range(3))
            f = DT * f * grp["ds"]
            self._back(y, grp["sides"][0], -f)
            self._back(y, grp["sides"][1], f)
        return y.reshape(-1)

    def solve(self, b, tol=1e-13, most=4000):
        """A^-1 b by CG with a diagonal preconditioner."""
        B2, D2 = (t * t for t in self.t)
        dg = _tp(self.m, B2.t(), B2.t(), B2.t())
        for d in range(3):
            kk = (self.Ji[:, d] ** 2).sum(1) * self.bw
            dg += _tp(kk, *[D2.t() if e == d else B2.t() for e in range(3)])
        dg = dg.reshape(-1)
        x, r = torch.zeros_like(b), b.clone()
        z = r / dg
        p, rz, stop = z.clone(), torch.dot(r, z), float(torch.linalg.norm(b)) * tol
        for it in range(most):
            q = self.apply(p)
            a = rz / torch.dot(p, q)
            x += a * p
            r -= a * q
            if it % 10 == 9 and float(torch.linalg.norm(r)) <= stop:
                return x
            z = r / dg
            new = torch.dot(r, z)
            p = z + new / rz * p
            rz = new
        return None


def _train_gradient(case, seed):
    """Gradient of mean((net(F) - T)^2) at the initial weights."""
    n = case["k"] + 1
    par, at = _network(case["k"], seed, 0.1).double(), 0
    g = _generator(seed, 3)
    n_in = n ** 3 + 6 * n * n + 1
    a = [torch.randn(case["batch"], n_in, dtype=torch.float32, device=DEV, generator=g).double()]
    T = torch.randn(case["batch"], n ** 3, dtype=torch.float32, device=DEV, generator=g).clamp_(-1, 1).double()
    W = []
    for l, (o, i) in enumerate(((256, n_in), (256, 256), (n ** 3, 256))):
        W.append(par[at:at + o * i].reshape(o, i))
        z = a[-1] @ W[-1].t() + par[at + o * i:at + o * i + o]
        at += o * i + o
        a.append(z.clamp_min(0) if l < 2 else z)
    d, grads = 2.0 * (a[3] - T) / T.numel(), []
    for l in (2, 1, 0):
        grads = [(d.t() @ a[l]).reshape(-1), d.sum(0)] + grads
        d = (d @ W[l]) * (a[l] > 0)
    return torch.cat(grads)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _train_gradient(case, seed)
    n = case["k"] + 1
    dofs = case["nx"] * case["ny"] * case["nz"] * n ** 3
    if kind in ("cg", "fgmres", "learned", "multigrid") and dofs > 6e5:
        return None      # its plain solve takes too long
    E = _Exact(case, 2 * case["k"] + 1 if kind == "consistent" else None)
    xyz = E.dofs()
    alpha, beta = _coefficients(xyz, case, _generator(seed, 1))
    g = _generator(seed, 2)
    b = _smooth(xyz, case, g)
    if kind == "pressure":
        return E.pressure(b, *_pressure_fields(xyz, case, _generator(seed, 1)))
    E.set(alpha, beta)
    if kind == "apply":
        return E.apply(b.float() if case["f32"] else b)
    if kind == "consistent":
        return E.apply(b)
    if kind in ("residual", "coefficients"):
        return b - E.apply(_smooth(xyz, case, g))
    return E.solve(b)

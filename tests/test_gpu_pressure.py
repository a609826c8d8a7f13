"""The pressure system of one IMEX stage on the GPU (section 2: A U + B P = F,
C U + D P = G, solved as S P = (D - C A^-1 B) P = G - C A^-1 F) against the
oracle's composition of its own B, C, A^-1 and D (pinned in
test_schur_oracle.py): every part, the system, the right-hand side and the
velocity recovery, on the tiny meshes at k = 1, 2, the terrain channel at
k = 4 and curved cells at k = 3; then FGMRES on S with the paper's
preconditioners (Helmholtz and internal-energy diagonals), block Jacobi and
the inner FP32 CG on the Helmholtz-type operator, each reaching the true
residual bar, with the solution compared to the oracle's."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from helpers import TINY, constructed_pressure_state, oracle_fixed_point, to_dev
from oracle.core import PressureSystem

pytestmark = pytest.mark.gpu

GAMMA, TAU = 1.4, 0.3


def _hx():
    import paper_2505_00384_amd as hx
    return hx


def _fields(p, name):
    x, y, z = p.dof_coords()
    if name.startswith("terrain"):
        rho, h = si.terrain_pressure_fields()
        return rho(x, y, z), h(x, y, z), si.TERRAIN["dt"]
    fr, _ = si.random_smooth_coefficients(3)
    fh, _ = si.random_smooth_coefficients(4)
    return fr(x, y, z), fh(x, y, z), TAU


def _setup(name, mk, k):
    m = mk()
    p = oracle.Problem(m, k)
    rho, h, tau = _fields(p, name)
    ref = PressureSystem(m, k, rho, h, GAMMA, tau)
    hx = _hx()
    ctx = hx.HelmDG(0)
    ctx.setup_mesh(k, p.nodes, p.nbr, p.g)
    ctx.set_pressure_system(rho, h, GAMMA, tau)
    return p, ref, ctx


def _close(a, b, tol, floor=0.0):
    """max|a - b| <= tol * max(max|b|, floor): the floor is the size of the
    individual terms where the result itself can vanish (on one periodic cell
    of degree 1 the central-flux gradient of every field is zero)."""
    a = np.asarray(a).ravel(); b = np.asarray(b).ravel()
    return np.abs(a - b).max() <= tol * max(np.abs(b).max(), floor)


CASES = [(name, mk, k) for (name, mk) in TINY for k in (1, 2)] + [
    ("terrain-4x2x3-g4", lambda: si.terrain_mesh(4, 2, 3, g=4), 4),
    ("wavy-2-g3", lambda: si.wavy_cube_mesh(2, 3), 3),
    ("terrain-3x2x2-g4", lambda: si.terrain_mesh(3, 2, 2, g=4), 6),
]


@pytest.mark.parametrize("name,mk,k", CASES, ids=[f"{c[0]}-k{c[2]}" for c in CASES])
def test_parts_match_oracle(name, mk, k):
    hx = _hx()
    print(f"[pressure] {name} k={k}", flush=True)
    p, ref, ctx = _setup(name, mk, k)
    n = p.n_dofs
    pv = si.random_vector(n, 21)
    u3 = si.random_vector(3 * n, 22).reshape(3, n)
    area = p.cell_volumes().max() ** (2.0 / 3.0) / (k + 1) ** 2   # a face quadrature weight
    tau = ref.tau
    g = ctx.apply_pressure_part(hx.HX_PS_GRAD, to_dev(pv)).cpu().numpy()
    assert _close(g, ref.grad(pv), 1e-12, tau * np.abs(pv).max() * area), "B"
    d = ctx.apply_pressure_part(hx.HX_PS_DIV, to_dev(u3)).cpu().numpy()
    assert _close(d, ref.div(u3), 1e-12, tau * np.abs(ref.hr).max() * np.abs(u3).max() * area), "C"
    ai = ctx.apply_pressure_part(hx.HX_PS_VMASS_INV, to_dev(u3)).cpu().numpy()
    assert _close(ai, ref.a_inv(u3), 1e-11), "A^-1"
    dm = ctx.apply_pressure_part(hx.HX_PS_DMASS, to_dev(pv)).cpu().numpy()
    assert _close(dm, ref.d_apply(pv), 1e-12), "D"
    s = ctx.apply_pressure_part(hx.HX_PS_SYSTEM, to_dev(pv)).cpu().numpy()
    assert _close(s, ref.apply(pv), 1e-11), "S"
    G = si.random_vector(n, 23)
    r = ctx.pressure_rhs(to_dev(u3), to_dev(G)).cpu().numpy()
    assert _close(r, ref.rhs(u3, G), 1e-11), "rhs"
    U = ctx.pressure_velocity(to_dev(u3), to_dev(pv)).cpu().numpy()
    assert _close(U, ref.velocity(u3, pv), 1e-11), "velocity"
    ctx.close()


def test_pressure_solves_terrain():
    """FGMRES on S with each preconditioner; the true residual of the GPU
    system decides, the oracle's residual of the same x confirms it, and the
    solutions agree with the oracle's 1e-12 solve."""
    hx = _hx()
    name, mk, k = "terrain-8x2x4-g4", (lambda: si.terrain_mesh(8, 2, 4, g=4)), 4
    p, ref, ctx = _setup(name, mk, k)
    n = p.n_dofs
    x, y, z = p.dof_coords()
    F = np.stack([si.rhs_terrain(s)(x, y, z) for s in (31, 32, 33)])
    G = si.rhs_terrain(34)(x, y, z)
    b = ref.rhs(F, G)
    # oracle reference with the inverse Helmholtz diagonal as preconditioner
    helm = oracle.Problem(p.mesh, k, alpha=np.full(n, 1.0 / (GAMMA - 1.0)),
                          beta=si.TERRAIN["dt"] ** 2 * _fields(p, name)[1])
    dinv = 1.0 / helm.cell_diagonal(stiff=True)
    xs, oi = oracle.solvers.fgmres(ref.apply, b, precond=lambda v: dinv * v, restart=30,
                                   rtol=1e-12, max_iter=5000)
    assert oi.converged
    bd = ctx.pressure_rhs(to_dev(F), to_dev(G))
    assert _close(bd.cpu().numpy(), b, 1e-11)
    its = {}
    for label, kw in [("helmholtz-diag", dict(pc=hx.HX_PC_HELMHOLTZ_DIAG)),
                      ("mass-diag", dict(pc=hx.HX_PC_MASS_DIAG)),
                      ("block-jacobi", dict(pc=hx.HX_PC_BLOCK_JACOBI)),
                      ("inner-cg", dict(pc=hx.HX_PC_BLOCK_JACOBI, mixed=1, inner_iters=8,
                                        restart=10))]:
        prm = hx.default_params(method=1, system=1, rtol=1e-8, max_iter=5000, **kw)
        xg, info = ctx.solve(bd, params=prm)
        print(f"[pressure] {label}: {info['iters']} it ({info['inner_iters']} inner), "
              f"{info['ms_total']:.1f} ms, res {info['true_rel_res']:.2e}", flush=True)
        assert info["status"] == hx.HX_OK and info["true_rel_res"] <= 1e-8, (label, info)
        xh = xg.cpu().numpy()
        assert np.linalg.norm(b - ref.apply(xh)) <= 1.01e-8 * np.linalg.norm(b) * 1.001 + \
            1e-12 * np.linalg.norm(b), label
        assert np.linalg.norm(xh - xs) <= 1e-6 * np.linalg.norm(xs), label
        its[label] = info["iters"]
    # the paper's Helmholtz diagonal beats the internal-energy diagonal
    assert its["helmholtz-diag"] < its["mass-diag"]
    U = ctx.pressure_velocity(to_dev(F), to_dev(xs)).cpu().numpy()
    assert _close(U, ref.velocity(F, xs), 1e-11)
    ctx.close()


def test_pressure_system_errors():
    hx = _hx()
    import torch
    m = si.cube_mesh(2)
    p = oracle.Problem(m, 1)
    ctx = hx.HelmDG(0)
    ctx.setup_mesh(1, p.nodes, p.nbr, p.g)
    v = torch.zeros(p.n_dofs, dtype=torch.float64, device="cuda:0")
    with pytest.raises(hx.HXError) as e:
        ctx.apply_pressure_part(hx.HX_PS_SYSTEM, v)
    assert e.value.status == hx.HX_ERR_STATE
    with pytest.raises(hx.HXError) as e:
        ctx.set_pressure_system(np.ones(p.n_dofs), np.ones(p.n_dofs), 1.0, 0.1)
    assert e.value.status == hx.HX_ERR_ARG
    ctx.set_pressure_system(np.ones(p.n_dofs), np.ones(p.n_dofs), GAMMA, 0.1)
    b = torch.ones(p.n_dofs, dtype=torch.float64, device="cuda:0")
    with pytest.raises(hx.HXError) as e:
        ctx.solve(b, params=hx.default_params(method=0, system=1))
    assert e.value.status == hx.HX_ERR_ARG
    with pytest.raises(hx.HXError) as e:
        ctx.apply_pressure_part(7, v)
    assert e.value.status == hx.HX_ERR_ARG
    ctx.close()


def test_fixed_point_recovers_constructed_state():
    """G is built so that a perturbed hydrostatic pressure p* is the fixed
    point; the GPU loop started from the unperturbed background converges to
    it, and its first two iterates equal the oracle's."""
    hx = _hx()
    m = si.terrain_mesh(4, 2, 3, g=4)
    k = 4
    p_or = oracle.Problem(m, k)
    rho, F, G, p_bg, p_star, tau = constructed_pressure_state(m, k, GAMMA)
    ctx = hx.HelmDG(0)
    ctx.setup_mesh(k, p_or.nodes, p_or.nbr, p_or.g)
    prm = hx.default_params(method=1, restart=30, rtol=1e-13, pc=hx.HX_PC_HELMHOLTZ_DIAG,
                            max_iter=5000)
    # two iterations against the oracle's two
    pd = to_dev(p_bg)
    pd, info = ctx.solve_pressure_fixed_point(to_dev(rho), to_dev(F), to_dev(G), pd, GAMMA, tau,
                                              params=prm, max_fp_iters=2, fp_tol=1e-300,
                                              check=False)
    assert info["fp_iters"] == 2 and info["status"] == hx.HX_ERR_NOCONV
    p2 = oracle_fixed_point(m, k, rho, F, G, p_bg, GAMMA, tau, 2)
    assert np.linalg.norm(pd.cpu().numpy() - p2) <= 1e-10 * np.linalg.norm(p2)
    # to convergence
    pd = to_dev(p_bg)
    pd, info = ctx.solve_pressure_fixed_point(to_dev(rho), to_dev(F), to_dev(G), pd, GAMMA, tau,
                                              params=prm, max_fp_iters=30, fp_tol=1e-11)
    print(f"[pressure] fixed point: {info}", flush=True)
    assert info["status"] == hx.HX_OK and info["fp_iters"] < 30
    assert np.linalg.norm(pd.cpu().numpy() - p_star) <= 1e-9 * np.linalg.norm(p_star)
    ctx.close()


def test_sampled_parity_full_size_terrain():
    """At the 256x64x64 Q4 size (the benchmarked configuration) the oracle
    computes B, C and S on sampled cells only."""
    import torch
    hx = _hx()
    free = torch.cuda.mem_get_info()[0]
    if free < 100e9:
        pytest.skip("needs ~100 GB of device memory")
    print("[pressure] terrain 256x64x64 k=4, sampled cells", flush=True)
    m = si.terrain_mesh(256, 64, 64, g=4)
    p, ref, ctx = _setup("terrain-256x64x64-g4", lambda: m, 4)
    n, nd = p.n_dofs, p.nd
    pv = si.random_vector(n, 5)
    u3 = si.random_vector(3 * n, 6).reshape(3, n)
    area = p.cell_volumes().max() ** (2.0 / 3.0) / 25.0     # a face quadrature weight
    rng = np.random.default_rng(0)
    cells = np.unique(np.concatenate([rng.integers(0, m.n_cells, 24),
                                      [0, 255, 256 * 63, m.n_cells - 1]]))
    idx = (cells[:, None] * nd + np.arange(nd)[None, :]).ravel()
    g = ctx.apply_pressure_part(hx.HX_PS_GRAD, to_dev(pv))
    gs = g[:, torch.from_numpy(idx).to(g.device)].cpu().numpy().reshape(3, cells.size, nd)
    del g
    gr = ref.vel.grad_cells(pv, cells, ref.tau).transpose(1, 0, 2)
    assert _close(gs, gr, 1e-12, ref.tau * np.abs(pv).max() * area), "B"
    d = ctx.apply_pressure_part(hx.HX_PS_DIV, to_dev(u3))
    ds = d[torch.from_numpy(idx).to(d.device)].cpu().numpy().reshape(cells.size, nd)
    del d
    assert _close(ds, ref.vel.div_cells(u3, ref.hr, cells, ref.tau), 1e-12,
                  ref.tau * np.abs(ref.hr).max() * np.abs(u3).max() * area), "C"
    s = ctx.apply_pressure_part(hx.HX_PS_SYSTEM, to_dev(pv))
    ss = s[torch.from_numpy(idx).to(s.device)].cpu().numpy().reshape(cells.size, nd)
    del s
    assert _close(ss, ref.apply_cells(pv, cells), 1e-11), "S"
    ctx.close()


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
def test_system_on_affine_and_general_cells(k):
    """S at every degree on a ragged channel with both kinds of cells (the
    cells far from the ridge are affine, with their own form of the kernel;
    degree 1 treats every cell as general): against the oracle, and with every
    cell taken as general, to 1e-11 as the other checks of S (both sides round
    differently; S is a difference of its terms)."""
    hx = _hx()
    p, ref, ctx = _setup("terrain-7x1x3-g2", lambda: si.terrain_mesh(7, 1, 3, g=2), k)
    try:
        counts, _ = ctx.operator_info()
        assert 0 < counts["affine_cells"] < counts["cells"]
        x = si.random_vector(p.n_dofs, 70 + k)
        sr = ref.apply(x)
        s1 = ctx.apply_pressure_part(hx.HX_PS_SYSTEM, to_dev(x)).cpu().numpy()
        assert _close(s1, sr, 1e-11)
        ctx.set_cell_compression(False)
        s2 = ctx.apply_pressure_part(hx.HX_PS_SYSTEM, to_dev(x)).cpu().numpy()
        assert _close(s2, sr, 1e-11) and _close(s1, s2, 1e-11)
        ctx.set_cell_compression(True)
    finally:
        ctx.close()

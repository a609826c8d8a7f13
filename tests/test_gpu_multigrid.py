"""Geometric multigrid on the GPU (section 3.1: CG preconditioned by
geometric multigrid for the SPD systems, Chebyshev smoothing) against the
oracle's V-cycle (pinned in test_multigrid_oracle.py): the transfers on
their own, including a coarse cell with no children; one V-cycle through
three levels with the same Chebyshev intervals on both sides; CG with it
reaching the true-residual bar in the oracle's iteration count and far
below block Jacobi; and the error paths of the link."""
import numpy as np
import pytest

import synth_inputs as si
from helpers import gpu_context, problem, to_dev, terrain_hierarchy, oracle_levels
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu


def _hx():
    import paper_2505_00384_amd as hx
    return hx


def _gpu_levels(levels):
    """Contexts for the oracle levels, linked, with the same Chebyshev
    polynomials."""
    ctxs = [gpu_context(L.prob) for L in levels]
    for l, L in enumerate(levels):
        ctxs[l].set_chebyshev(L.degree, L.lo, L.hi)
        if l + 1 < len(levels):
            ctxs[l].set_multigrid(ctxs[l + 1], L.parent, L.octant)
    return ctxs


def _close(ctxs):
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("k", [1, 3, 4, 7])
def test_transfers_match_oracle(k):
    import torch
    fine = problem(si.terrain_mesh(6, 4, 2, g=2), k, coef="terrain")
    coarse = problem(si.terrain_mesh(3, 2, 1, g=2), k, coef="terrain")
    parent, octant = si.refinement_parents(3, 2, 1)
    cf, cc = gpu_context(fine), gpu_context(coarse)
    cf.set_multigrid(cc, parent, octant)
    r = si.random_vector(fine.n_dofs, 1)
    out = torch.full((coarse.n_dofs,), 7.0, dtype=torch.float64, device="cuda:0")
    cf.mg_transfer(0, to_dev(r), out)
    ref = mg.restrict(k, parent, octant, r, coarse.n_cells)
    err = np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()
    print(f"[mg] restrict k={k}: {err:.2e}", flush=True)
    assert err <= 1e-14
    xc = si.random_vector(coarse.n_dofs, 2)
    y0 = si.random_vector(fine.n_dofs, 3)
    y = to_dev(y0)
    cf.mg_transfer(1, to_dev(xc), y)
    ref = y0 + mg.prolong(k, parent, octant, xc)
    err = np.abs(y.cpu().numpy() - ref).max() / np.abs(ref).max()
    print(f"[mg] prolong k={k}: {err:.2e}", flush=True)
    assert err <= 1e-14
    _close([cf, cc])


def test_transfers_with_childless_coarse_cell():
    """Fine cells of a 4x2x2 box mapped into the first two cells of a 3x1x1
    box: the third coarse cell has no children (its restriction is zero)."""
    import torch
    k = 3
    fine = problem(si.box_mesh(4, 2, 2), k, coef="const")
    coarse = problem(si.box_mesh(3, 1, 1), k, coef="const")
    f = np.arange(16)
    fx, fy, fz = f % 4, (f // 4) % 2, f // 8
    parent = (fx // 2).astype(np.int32)
    octant = ((fx & 1) + 2 * fy + 4 * fz).astype(np.int32)
    cf, cc = gpu_context(fine), gpu_context(coarse)
    cf.set_multigrid(cc, parent, octant)
    r = si.random_vector(fine.n_dofs, 4)
    out = torch.full((coarse.n_dofs,), 7.0, dtype=torch.float64, device="cuda:0")
    cf.mg_transfer(0, to_dev(r), out)
    ref = mg.restrict(k, parent, octant, r, coarse.n_cells)
    o = out.cpu().numpy()
    assert np.abs(o - ref).max() <= 1e-14 * np.abs(ref).max()
    assert np.all(o[2 * 64:] == 0.0)
    _close([cf, cc])


@pytest.fixture(scope="module")
def hierarchy():
    probs, maps = terrain_hierarchy(8, 4, 4, 3, 4)
    return oracle_levels(probs, maps)


def test_vcycle_matches_oracle(hierarchy):
    hx = _hx()
    levels = hierarchy
    ctxs = _gpu_levels(levels)
    for seed in (5, 6):
        b = si.random_vector(levels[0].prob.n_dofs, seed)
        z = ctxs[0].apply_preconditioner(to_dev(b), kind=hx.HX_PC_MULTIGRID).cpu().numpy()
        ref = mg.vcycle(levels, b)
        err = np.abs(z - ref).max() / np.abs(ref).max()
        print(f"[mg] V-cycle seed {seed}: {err:.2e}", flush=True)
        assert err <= 1e-11
    # the FP32 cycle: the same V up to FP32 rounding
    b = si.random_vector(levels[0].prob.n_dofs, 5)
    z = ctxs[0].apply_preconditioner(to_dev(b), kind=hx.HX_PC_MULTIGRID_MIXED).cpu().numpy()
    ref = mg.vcycle(levels, b)
    err = np.abs(z - ref).max() / np.abs(ref).max()
    print(f"[mg] FP32 V-cycle: {err:.2e}", flush=True)
    assert err <= 2e-5
    # the middle level's own V-cycle (two levels) too
    b = si.random_vector(levels[1].prob.n_dofs, 7)
    z = ctxs[1].apply_preconditioner(to_dev(b), kind=hx.HX_PC_MULTIGRID).cpu().numpy()
    ref = mg.vcycle(levels[1:], b)
    assert np.abs(z - ref).max() <= 1e-11 * np.abs(ref).max()
    _close(ctxs)


def test_mg_cg_matches_oracle_iterations():
    hx = _hx()
    probs, maps = terrain_hierarchy(16, 4, 8, 3, 2)
    levels = oracle_levels(probs, maps)
    ctxs = _gpu_levels(levels)
    p = probs[0]
    bh = p.load_vector(si.rhs_terrain(0))
    x_ref, info_ref = mg.mg_cg(levels, bh, rtol=1e-8)
    x, info = ctxs[0].solve(to_dev(bh), params=hx.default_params(method=0, rtol=1e-8,
                                                                 pc=hx.HX_PC_MULTIGRID))
    _, i_bj = ctxs[0].solve(to_dev(bh), params=hx.default_params(method=0, rtol=1e-8))
    print(f"[mg] CG+MG {info['iters']} iterations (oracle {info_ref.iters}), block Jacobi "
          f"{i_bj['iters']}", flush=True)
    assert info["status"] == hx.HX_OK and info["true_rel_res"] <= 1e-8
    assert abs(info["iters"] - info_ref.iters) <= 1
    assert info["iters"] * 3 <= i_bj["iters"]
    xs = x.cpu().numpy()
    assert np.linalg.norm(xs - x_ref) <= 1e-6 * np.linalg.norm(x_ref)
    _close(ctxs)


def test_mg_cg_terrain_32x8x16_gpu_estimates():
    """The 32x8x16 Q4 terrain channel with four levels, the intervals from the
    library's own Lanczos estimates."""
    import torch
    hx = _hx()
    probs, maps = terrain_hierarchy(32, 8, 16, 4, 4)
    ctxs = [gpu_context(p) for p in probs]
    g = torch.Generator(device="cuda:0")
    for l, (c, p) in enumerate(zip(ctxs, probs)):
        g.manual_seed(10 + l)
        lo, hi = c.estimate_eigenvalues(torch.randn(p.n_dofs, dtype=torch.float64,
                                                    device="cuda:0", generator=g), 20)
        if l + 1 < len(ctxs):
            c.set_chebyshev(3, 1.1 * hi / 15.0, 1.1 * hi)
            c.set_multigrid(ctxs[l + 1], *maps[l])
        else:
            c.set_chebyshev(12, 0.9 * lo, 1.1 * hi)
    p = probs[0]
    b = to_dev(p.load_vector(si.rhs_terrain(0)))
    x, info = ctxs[0].solve(b, params=hx.default_params(method=0, rtol=1e-8, pc=hx.HX_PC_MULTIGRID))
    _, i_bj = ctxs[0].solve(b, params=hx.default_params(method=0, rtol=1e-8))
    print(f"[mg] 32x8x16: CG+MG {info['iters']} iterations {info['ms_total']:.1f} ms; block "
          f"Jacobi {i_bj['iters']} iterations {i_bj['ms_total']:.1f} ms", flush=True)
    assert info["status"] == hx.HX_OK and info["true_rel_res"] <= 1e-8
    assert info["iters"] <= 15 and info["iters"] * 4 <= i_bj["iters"]
    _, fi = ctxs[0].solve(b, params=hx.default_params(method=1, rtol=1e-8, pc=hx.HX_PC_MULTIGRID))
    assert fi["status"] == hx.HX_OK and fi["true_rel_res"] <= 1e-8
    # the FP32 cycle inside FP64 CG: the same iteration count within two
    xm, im = ctxs[0].solve(b, params=hx.default_params(method=0, rtol=1e-8,
                                                       pc=hx.HX_PC_MULTIGRID_MIXED))
    print(f"[mg] 32x8x16: CG + FP32 V-cycle {im['iters']} iterations {im['ms_total']:.1f} ms",
          flush=True)
    assert im["status"] == hx.HX_OK and im["true_rel_res"] <= 1e-8
    assert abs(im["iters"] - info["iters"]) <= 2
    assert float((xm - x).norm() / x.norm()) <= 1e-7
    _close(ctxs)


def test_multigrid_errors():
    hx = _hx()
    fine = problem(si.terrain_mesh(4, 2, 2, g=2), 2, coef="terrain")
    coarse = problem(si.terrain_mesh(2, 1, 1, g=2), 2, coef="terrain")
    other = problem(si.terrain_mesh(2, 1, 1, g=2), 3, coef="terrain")
    parent, octant = si.refinement_parents(2, 1, 1)
    cf, cc, co = gpu_context(fine), gpu_context(coarse), gpu_context(other)
    b = to_dev(si.random_vector(fine.n_dofs, 1))

    def status(fn):
        with pytest.raises(hx.HXError) as e:
            fn()
        return e.value.status
    assert status(lambda: cf.set_multigrid(co, parent, octant)) == hx.HX_ERR_ARG      # degree
    bad = octant.copy(); bad[1] = bad[0]
    assert status(lambda: cf.set_multigrid(cc, parent, bad)) == hx.HX_ERR_ARG         # octant twice
    bad = parent.copy(); bad[0] = 2
    assert status(lambda: cf.set_multigrid(cc, bad, octant)) == hx.HX_ERR_ARG         # no such parent
    cf.set_multigrid(cc, parent, octant)
    assert status(lambda: cc.set_multigrid(cf, np.zeros(2, np.int32), np.arange(2, dtype=np.int32))
                  ) == hx.HX_ERR_ARG                                                  # cycle
    # no smoothers yet
    assert status(lambda: cf.apply_preconditioner(b, kind=hx.HX_PC_MULTIGRID)) == hx.HX_ERR_STATE
    cf.set_chebyshev(2, 0.1, 2.0)
    assert status(lambda: cf.solve(b, params=hx.default_params(method=0, pc=hx.HX_PC_MULTIGRID))
                  ) == hx.HX_ERR_STATE                                                # coarse level
    cc.set_chebyshev(8, 0.01, 2.0)
    z = cf.apply_preconditioner(b, kind=hx.HX_PC_MULTIGRID)
    assert bool(z.isfinite().all())
    assert status(lambda: cf.solve(b, params=hx.default_params(method=1, mixed=1,
                                                              pc=hx.HX_PC_MULTIGRID))) == hx.HX_ERR_ARG
    assert status(lambda: cf.apply_preconditioner(b.float(), kind=hx.HX_PC_MULTIGRID)) == hx.HX_ERR_ARG
    assert status(lambda: cf.apply_preconditioner(b.float(), kind=hx.HX_PC_MULTIGRID_MIXED)
                  ) == hx.HX_ERR_ARG
    zm = cf.apply_preconditioner(b, kind=hx.HX_PC_MULTIGRID_MIXED)
    assert float((zm - z).norm() / z.norm()) <= 1e-5
    # the coarse level set up again: the link must be set again
    cc.setup_mesh(coarse.k, coarse.nodes, coarse.nbr, coarse.g)
    cc.set_coefficients(coarse.alpha, coarse.beta, coarse.P)
    cc.set_chebyshev(8, 0.01, 2.0)
    assert status(lambda: cf.apply_preconditioner(b, kind=hx.HX_PC_MULTIGRID)) == hx.HX_ERR_STATE
    cf.set_multigrid(cc, parent, octant)
    cf.apply_preconditioner(b, kind=hx.HX_PC_MULTIGRID)
    # closing the coarse level removes the link
    cc.close()
    assert status(lambda: cf.mg_transfer(0, b, b.clone())) == hx.HX_ERR_STATE
    _close([cf, co])


@pytest.mark.parametrize("mesh,k", [(m, k) for m in ("terrain", "general", "cube") for k in range(1, 8)]
                         + [("large", 4), ("large", 6)])
def test_single_precision_smoothing_steps(mesh, k):
    """The FP32 cycle, whose smoothing steps are one launch each on two
    buffers in turn, against the FP64 cycle of the same levels: Chebyshev
    degrees of both parities (from zero and from a given iterate), on meshes
    with affine and general cells, general ones only and affine ones only, and
    on one with more than 1024 workgroups (the operator's one-wave form).
    Tolerance: 2e-6 per FP32 operator application (its own test), at most 18
    of them, times 5 for the cell solves: 2e-4; a step on the wrong iterate is
    off by 1e-2 and more."""
    hx = _hx()
    if mesh == "cube":
        fine, coarse = si.cube_mesh(4), si.cube_mesh(2)
        parent, octant = si.refinement_parents(2, 2, 2)
        coef = "const"
    else:
        nx, ny, nz = (22, 4, 3) if mesh == "large" else (7, 1, 3)
        fine, coarse = si.terrain_mesh(2 * nx, 2 * ny, 2 * nz, g=2), si.terrain_mesh(nx, ny, nz, g=2)
        parent, octant = si.refinement_parents(nx, ny, nz)
        coef = "terrain"
    ctxs = [gpu_context(problem(m, k, coef=coef)) for m in (fine, coarse)]
    try:
        b = [to_dev(si.random_vector(c.n_dofs, 90 + k)) for c in ctxs]
        for c in ctxs:
            c.set_cell_compression(mesh != "general")
        bounds = [c.estimate_eigenvalues(v, 15) for c, v in zip(ctxs, b)]
        ctxs[0].set_multigrid(ctxs[1], parent, octant)
        for degree in (1, 2, 3, 4):
            print(f"[mg32] {mesh} k={k} degree={degree}", flush=True)
            for c, (lo, hi) in zip(ctxs, bounds):
                c.set_chebyshev(degree, 1.1 * hi / 15.0, 1.1 * hi)
            z = [ctxs[0].apply_preconditioner(b[0], kind=kind).cpu().numpy()
                 for kind in (hx.HX_PC_MULTIGRID, hx.HX_PC_MULTIGRID_MIXED)]
            assert np.linalg.norm(z[1] - z[0]) <= 2e-4 * np.linalg.norm(z[0])
    finally:
        _close(ctxs)

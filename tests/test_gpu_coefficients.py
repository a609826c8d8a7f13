"""The coefficient update: its two forms (compressed data in use, or the
general data written for every cell), the general data rebuilt from the
compressed ones on request, and the face constants after a change of the
penalty, on a mesh with affine and general cells (a terrain channel whose
cells far from the ridge are affine) and a ragged cell count.

Tolerances: operator against the oracle 1e-12 (as in the parity tests); the
rebuilt general values differ from the directly merged ones only by the
rounding of a product and of J^-1 J^-T, taken per cell or per point: 1e-13 of
the largest value."""
import numpy as np
import pytest

import synth_inputs as si
from helpers import gpu_context, problem, to_dev, normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
def test_forms_of_the_coefficient_update(k):
    import paper_2505_00384_amd as hx
    p = problem(si.terrain_mesh(7, 1, 3, g=2), k, coef="terrain")
    n = k + 1
    nc, nd, nf = p.n_cells, n ** 3, n * n
    x = si.random_vector(p.n_dofs, 60 + k)
    ref = p.apply(x)
    ctx = gpu_context(p)
    try:
        counts, _ = ctx.operator_info()
        print(f"[coef] k={k} {counts}", flush=True)
        assert 0 < counts["affine_cells"] < counts["cells"] and counts["affine_faces"] > 0

        def apply():
            y = ctx.apply_operator(to_dev(x)).cpu().numpy()
            assert max(normwise(y, ref)) <= 1e-12

        def export():
            return (ctx.debug_export(hx.HX_EXPORT_CELL_DATA, (nc, 7, nd)),
                    ctx.debug_export(hx.HX_EXPORT_FACE_DATA, (nc, 3, 7, nf)),
                    ctx.debug_export(hx.HX_EXPORT_INV_DIAG, (2, p.n_dofs)))

        apply()                                    # compressed
        lean = export()                            # general data rebuilt
        ctx.set_cell_compression(False)
        apply()
        ctx.set_coefficients(p.alpha, p.beta, p.P)  # general data written
        apply()
        full = export()
        for a, b in zip(lean, full):
            assert np.abs(a - b).max() <= 1e-13 * np.abs(b).max()
        ctx.set_cell_compression(True)
        apply()                                    # compressed data written by that update too
        # other coefficients and another penalty, compressed, then the
        # compression off without an update in between
        q = problem(si.terrain_mesh(7, 1, 3, g=2), k, coef="random", seed=k, P=3.0)
        ctx.set_coefficients(q.alpha, q.beta, q.P)
        ref = q.apply(x)
        apply()
        ctx.set_cell_compression(False)
        apply()
        y32 = ctx.apply_operator(to_dev(x.astype(np.float32))).cpu().numpy()
        assert normwise(y32, ref)[0] <= 2e-6
    finally:
        ctx.close()


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
def test_single_precision_face_data(k):
    """The FP32 face data have an order of their own up to degree 6: the FP32
    operator with compressed data, with general data written by the update and
    with general data rebuilt from the compressed ones.  Tolerance 2e-6, as for
    the FP32 operator above (rounded data and about 3 (k + 1) roundings a
    sweep, 6e-8 each)."""
    p = problem(si.terrain_mesh(7, 1, 3, g=2), k, coef="terrain")
    x = si.random_vector(p.n_dofs, 80 + k)
    ref = p.apply(x)
    ctx = gpu_context(p)
    try:
        def apply(what):
            print(f"[coef32] k={k} {what}", flush=True)
            y = ctx.apply_operator(to_dev(x.astype(np.float32))).cpu().numpy()
            assert normwise(y, ref)[0] <= 2e-6, what

        apply("compressed")
        ctx.set_cell_compression(False)
        apply("rebuilt")
        ctx.set_coefficients(p.alpha, p.beta, p.P)
        apply("written")
    finally:
        ctx.close()

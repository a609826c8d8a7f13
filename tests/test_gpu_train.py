"""A training step (forward, back-propagated signals, weight and bias
gradients, Adam) at the edges of its tiles: batches around the 16-row
workgroups, the 32-row steps and the 256-row chunks of the weight gradient,
more than 16 chunks, and the smallest and largest degrees.

Tolerance: every product is checked on the operands the GPU used (exported by
the trace), so only the FP32 accumulation differs from the FP64 reference:
its relative error is at most about sqrt(K) 2^-24 for K = 897 or 4,097
random-sign terms, 4e-6; 1e-5 normwise per block, as for the whole step's
other layer checks."""
import numpy as np
import pytest

import synth_inputs as si
from helpers import gpu_context, problem, to_dev
from oracle import mlp

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300)


@pytest.mark.parametrize("k,B", [(1, 1), (1, 33), (2, 16), (2, 257), (3, 31), (4, 17), (4, 32),
                                 (4, 4097), (5, 255), (6, 48), (7, 65)])
def test_training_step_at_tile_edges(k, B):
    import paper_2505_00384_amd as hx
    print(f"[train] k={k} B={B}", flush=True)
    ctx = gpu_context(problem(si.cube_mesh(2), k, coef="const"))
    try:
        n = k + 1
        n_in, n_out = n ** 3 + 6 * n * n + 1, n ** 3
        w = si.mlp_init(21, n_in=n_in, n_out=n_out)
        w[-n_out:] = 0.02
        ctx.set_network(w)
        rng = np.random.default_rng(100 * k + B)
        X = rng.normal(size=(B, n_in)).astype(np.float32)
        T = rng.normal(size=(B, n_out)).astype(np.float32)
        loss, g = ctx.train_step(to_dev(X), to_dev(T), 1e-3, want_grad=True)
        g = g.cpu().numpy().astype(np.float64)
        tr = {t: ctx.network_trace(getattr(hx, "HX_TRACE_" + t), B).astype(np.float64)
              for t in ("INPUT", "H1", "H2", "OUT", "DOUT", "DH2", "DH1")}
        o = 0
        W = []
        for rows, cols in ((256, n_in), (256, 256), (n_out, 256)):
            W.append((w[o:o + rows * cols].astype(np.float64).reshape(rows, cols),
                      w[o + rows * cols:o + rows * (cols + 1)].astype(np.float64)))
            o += rows * (cols + 1)
        rb, tol = mlp.bf16_round, 1e-5
        np.testing.assert_array_equal(tr["INPUT"], rb(X))
        assert _rel(tr["H1"], np.maximum(mlp.layer(*W[0], tr["INPUT"]), 0)) <= tol
        assert _rel(tr["H2"], np.maximum(mlp.layer(*W[1], rb(tr["H1"])), 0)) <= tol
        assert _rel(tr["OUT"], mlp.layer(*W[2], rb(tr["H2"]))) <= tol
        assert _rel(tr["DOUT"], 2.0 * (tr["OUT"] - T) / T.size) <= tol
        assert abs(loss - np.mean((tr["OUT"] - T) ** 2)) <= 1e-5 * loss
        blocks, back = [], None
        for l, d, a, h in ((2, "DOUT", "H2", "DH2"), (1, "DH2", "H1", "DH1"), (0, "DH1", "INPUT", None)):
            gW, gb, back = mlp.layer_grads(W[l][0], tr[d], rb(tr[a]))
            blocks = [gW.ravel(), gb] + blocks
            if h:
                assert _rel(tr[h], back * (tr[a] > 0)) <= tol, h
        o = 0
        for i, blk in enumerate(blocks):
            assert _rel(g[o:o + blk.size], blk) <= tol, i
            o += blk.size
        assert o == g.size
        # the Adam step, and the BF16 copies that the next forward passes read:
        # the batched one (row-major) and the training one (fragments)
        w1 = ctx.get_network()
        ref, _, _ = mlp.adam_step(w.astype(np.float64), g, 0.0, 0.0, 1, 1e-3)
        np.testing.assert_allclose(w1, ref, rtol=0, atol=2e-6)
        out = ctx.network_forward(to_dev(X)).cpu().numpy()
        ctx.train_step(to_dev(X), to_dev(T), 0.0)
        np.testing.assert_array_equal(ctx.network_trace(hx.HX_TRACE_OUT, B), out)
        # and the fragments of a network loaded afresh equal those kept by the update
        ctx.set_network(w1)
        ctx.train_step(to_dev(X), to_dev(T), 0.0)
        np.testing.assert_array_equal(ctx.network_trace(hx.HX_TRACE_OUT, B), out)
    finally:
        ctx.close()

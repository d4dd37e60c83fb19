"""Training gradients at the edges of the kernels' tiles: batches of one row to
several splits, ragged last tiles, widths with and without the row-tile kernel,
operands whose rows are not 16-byte aligned, more roots than lanes of a
half-wave; and the transposed weight copies after optimiser steps."""
import numpy as np
import pytest

from oracle import mlp_oracle as MO

pytestmark = pytest.mark.gpu


def _weights(rng, dims):
    return np.concatenate([np.r_[rng.uniform(-1, 1, (o, i)).ravel() * np.sqrt(3.0 / i), 0.1 * rng.standard_normal(o)]
                           for i, o in zip(dims[:-1], dims[1:])]).astype(np.float32)


def _inputs(rng, B, din, R):
    import torch

    X = torch.as_tensor(rng.standard_normal((B, din)).astype(np.float32), device="cuda").to(torch.bfloat16)
    roots = rng.uniform(0, 2 * np.pi, (B, R)).astype(np.float32)
    nroots = rng.integers(0, R + 1, B).astype(np.int32)
    return X, torch.as_tensor(roots, device="cuda"), torch.as_tensor(nroots, device="cuda")


@pytest.mark.parametrize("B,din,width,dout,R", [
    (1, 70, 256, 24, 6),        # one row
    (33, 118, 256, 40, 32),     # one row past a tile, rows of 236 bytes
    (65, 9, 32, 2, 5),          # odd input width, the smallest outputs
    (700, 255, 224, 48, 40),    # several splits, the last ragged; more than 32 roots
    (40, 300, 256, 24, 8),      # inputs past the row-tile kernel: one GEMM per layer
    (300, 22, 48, 8, 16),       # width not a multiple of 32
    (70, 33, 320, 6, 9),        # width past the row-tile kernel
])
def test_gradients_at_tile_edges(B, din, width, dout, R):
    import paper_2101_12348_amd as F

    rng = np.random.default_rng(B + din)
    dims = [din, width, width, width, dout]
    w = _weights(rng, dims)
    net = F.Mlp(din, width, dout, weights=w)
    X, roots, nroots = _inputs(rng, B, din, R)
    loss, grads = net.loss_grad(X, roots, nroots, lam=0.5)
    out = net.forward(X).cpu().numpy().astype(np.float64)
    p, o = {}, 0
    for l in range(4):
        i, n = dims[l], dims[l + 1]
        p["W" + MO.LAYER_NAMES[l]] = w[o:o + i * n].reshape(n, i).astype(np.float64)
        o += i * n
        p["b" + MO.LAYER_NAMES[l]] = w[o:o + n].astype(np.float64)
        o += n
    _, cache = MO.forward(p, X.float().cpu().numpy().astype(np.float64), emulate_bf16=True)
    L, dref = MO.chamfer_loss(out, roots.cpu().numpy().astype(np.float64), nroots.cpu().numpy(), lam=0.5)
    ref = MO.backward(p, cache, dref, emulate_bf16=True)
    assert abs(float(loss.double().mean()) - L) <= 1e-4 * max(1.0, abs(L))
    g, o = grads.cpu().numpy().astype(np.float64), 0
    for k in MO.LAYER_NAMES:
        for name in ("W" + k, "b" + k):
            r = ref[name].ravel()
            # bf16 operands: a rounding near a tie may differ from the reference's by one step (2^-8)
            assert np.max(np.abs(g[o:o + r.size] - r)) <= 3e-2 * max(np.max(np.abs(r)), 1e-12), name
            o += r.size


@pytest.mark.parametrize("width", [256, 96])
def test_transposed_weights_follow_the_optimiser(width):
    import torch
    import paper_2101_12348_amd as F

    rng = np.random.default_rng(width)
    din, dout = 118, 40
    net = F.Mlp(din, width, dout, weights=_weights(rng, [din, width, width, width, dout]))
    X, roots, nroots = _inputs(rng, 200, din, 12)
    for _ in range(3):
        net.train_step(X, roots, nroots, lr=1e-2)
    fresh = F.Mlp(din, width, dout, weights=net.weights())
    a, b = net.loss_grad(X, roots, nroots), fresh.loss_grad(X, roots, nroots)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])

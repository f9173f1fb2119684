"""Training step against the oracle at the edges of its tiles: 64 rows a tile,
one tile a block up to 256 tiles, then several; and inference over many tiles."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import pairgen
from oracle import mlp as om

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    """Rows of the model's 64 inputs: m / 512, E / 32 and shares of matching cells."""
    rng = np.random.default_rng(seed)
    X = np.zeros((n, 64), np.float32)
    X[:, 0] = rng.choice([64, 100, 150, 250, 300], n) / 512
    X[:, 1] = rng.integers(3, 16, n) / 32
    X[:, 17:48] = rng.integers(0, 65, (n, 31)) / 64
    return X, rng.integers(0, 33, n).astype(np.float32)


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 16384, 16385, 40000])
def test_step_at_tile_edges(gpu_ctx, n):
    p = pairgen.init_mlp_params(11)
    gpu_ctx.mlp_set_params(p)
    X, t = _rows(n, n)
    loss, grads = gpu_ctx.mlp_train_step(torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda(), lr=0.0, want_grads=True)
    w = om.working_weights(p)
    ref_loss, g = om.loss_and_grads(w, om.bf16_round(X), t)
    gd = om.unpack(grads.cpu().numpy().astype(np.float64))
    # Activations and gradients are rounded to bf16 (2^-9 each) at four places on the way.
    tol = 4 * 2.0 ** -8
    assert abs(loss.item() - ref_loss) <= tol * ref_loss
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        assert _rel(gd[k], g[k]) <= tol, (k, _rel(gd[k], g[k]))
    y = gpu_ctx.mlp_forward(torch.from_numpy(X).cuda()).cpu().numpy()
    e = (y.astype(np.float64) - t)
    # the loss and the predictions come from the same forward pass
    assert abs(np.mean(e * e) - loss.item()) <= 1e-5 * ref_loss

"""Inference over more rows than one launch holds: the first and last rows of
every launch, and the rows between, against the same rows in a call of their
own (a row's prediction does not depend on the others)."""
from __future__ import annotations

import pytest
import torch

import pairgen

pytestmark = pytest.mark.gpu

LAUNCH_ROWS = 1 << 28


def test_more_rows_than_a_launch(gpu_ctx):
    n = 2 * LAUNCH_ROWS + 65
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < n * 64 * 4 + (8 << 30):
        pytest.skip("not enough free device memory for 2^29 rows")
    gpu_ctx.mlp_set_params(pairgen.init_mlp_params(17))
    gen = torch.Generator(device="cuda").manual_seed(1)
    at = torch.cat([torch.arange(a, b, device="cuda") for a, b in
                    ((0, 65), (LAUNCH_ROWS - 64, LAUNCH_ROWS + 65), (2 * LAUNCH_ROWS - 64, n))])
    rows = torch.rand((at.numel(), 64), generator=gen, device="cuda")
    X = torch.zeros((n, 64), dtype=torch.float32, device="cuda")
    X[at] = rows
    y = gpu_ctx.mlp_forward(X)
    del X
    want = gpu_ctx.mlp_forward(rows)
    zero = gpu_ctx.mlp_forward(torch.zeros((1, 64), device="cuda"))
    assert torch.equal(y[at], want)
    y[at] = zero
    assert bool((y == zero).all())
    gpu_ctx.check()
    del y
    torch.cuda.empty_cache()

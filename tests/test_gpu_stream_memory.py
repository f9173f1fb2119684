"""Streamed batches whose buffers do not fit next to the shapes of earlier ones:
a batch of few long pairs, then one of many short ones on the same context, with
the device's memory free and with little of it left."""
from __future__ import annotations

import pytest
import torch

import paper_1910_03936_amd as paf

pytestmark = pytest.mark.gpu
SS = paf.SNEAKYSNAKE
LONG, SHORT = 3_500_032, 32_000_000   # pairs of 512 and of 32 bases


def _zeros(n, m):
    """n pairs of m times base A: every pair equal, none rejected."""
    words = n * paf.words_for(m)
    return paf.HostBatch(torch.zeros(words, dtype=torch.int64), torch.zeros(words, dtype=torch.int64),
                         torch.full((n,), m, dtype=torch.int16), torch.zeros(n, dtype=torch.uint8), m, 0)


def _run(ctx, n, m):
    out, _ = paf.stream_filter(ctx, _zeros(n, m), (n + 63) // 64 * 64, SS)
    assert int(out[SS][1].max()) == 0
    assert int(paf.accept_bits_to_bool(out[SS][0], n).sum()) == n


def _free():
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("left", [None, 128 << 20])
def test_shapes_that_do_not_fit_together(left):
    torch.cuda.empty_cache()
    ctx = paf.Context(0)
    before = _free()
    _run(ctx, LONG, 512)
    kept = before - _free()
    assert 1_800_000_000 < kept < (2 << 30) + (64 << 20)
    # Room for the second batch's buffers once the first one's are gone, not for both shapes'.
    filler = None if left is None else torch.empty(_free() - left, dtype=torch.uint8, device="cuda")
    _run(ctx, SHORT, 32)
    if left is None:
        assert 1_800_000_000 < before - _free() < (2 << 30) + (64 << 20)
    del filler
    torch.cuda.empty_cache()
    _run(ctx, 1000, 32)
    ctx.check()
    ctx.close()
    assert before - _free() < 64 << 20

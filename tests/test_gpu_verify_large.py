"""Verification of batches large enough that a wave lists several tiles and its
lanes take new pairs as they finish: every pair selected, the survivors of
SneakySnake and a sparse selection, uniform and per-pair lengths with offsets,
a thresholds' violation in the middle of a list; whole numbers against the
oracle on a sample, and on every pair against the result without a selection."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import pairgen
import paper_1910_03936_amd as paf
from gpu_util import to_device

pytestmark = pytest.mark.gpu
SS = paf.SNEAKYSNAKE


def _dist(t):
    torch.cuda.synchronize()
    return paf.counts_u16(t).cpu().numpy().astype(np.int64)


@pytest.mark.parametrize("uneven,n", [(False, 64 * 3072 * 2 + 7), (True, 64 * 3072 + 65)])
def test_refilled_lanes(gpu_ctx, uneven, n):
    w = pairgen.UNEVEN_MIX if uneven else pairgen.FIXED_250BP.with_E(10)
    p = pairgen.generate(w, 0, n)
    b = to_device(p, gpu_ctx, per_pair=uneven, offsets=uneven)
    every = _dist(gpu_ctx.verify(b))
    E = p.E.astype(np.int64)
    assert np.all((every >= 0) & (every <= E + 1))
    ids = pairgen.sample_ids(n, 8000)
    want = oracle.banded_batch(p.reads[ids], p.refs[ids], p.len[ids], p.E[ids]).astype(np.int64)
    assert np.array_equal(every[ids], want)
    # SneakySnake rejects no pair within E edits.
    assert np.array_equal(_dist(gpu_ctx.verify(b, gpu_ctx.filter(b, SS)[SS][0])), every)
    bits = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    bits[::7] = 1 << 5
    sel = np.zeros(n, bool)
    sel[5::224] = True
    assert np.array_equal(_dist(gpu_ctx.verify(b, bits)), np.where(sel, every, E + 1))
    gpu_ctx.check()


def test_violation_inside_a_list(gpu_ctx):
    n = 64 * 3072 + 100
    p = pairgen.generate(pairgen.UNEVEN_MIX, 0, n)
    E = p.E.copy()
    E[70_001] = 20
    q = pairgen.Pairs(p.reads, p.refs, p.len, E, p.related, p.k)
    got = _dist(gpu_ctx.verify(to_device(q, gpu_ctx, per_pair=True, offsets=True, max_E=15)))
    with pytest.raises(paf.PafError):
        gpu_ctx.check()
    good = _dist(gpu_ctx.verify(to_device(p, gpu_ctx, per_pair=True, offsets=True, max_E=15)))
    good[70_001] = 0
    assert np.array_equal(got, good)
    gpu_ctx.check()


def test_lists_of_more_than_32_tiles(gpu_ctx):
    # One small batch over and over (its rows repeated on the device), so many
    # pairs that a wave lists more than 2048 of them; the repeats' distances
    # are the small batch's.
    base = 64 * 512
    p = pairgen.generate(pairgen.FIXED_250BP.with_E(25), 11, base)
    b = to_device(p, gpu_ctx, per_pair=False, offsets=False)
    times = 120
    n = base * times
    big = paf.Batch(reads=b.reads.repeat(times, 1) if b.reads.dim() > 1 else b.reads.repeat(times),
                    refs=b.refs.repeat(times, 1) if b.refs.dim() > 1 else b.refs.repeat(times),
                    n_pairs=n, stride_words=b.stride_words, uniform_len=b.uniform_len, uniform_E=b.uniform_E,
                    max_len=b.max_len, max_E=b.max_E)
    want = oracle.banded_batch(p.reads, p.refs, p.len, p.E).astype(np.int64)
    got = _dist(gpu_ctx.verify(big, gpu_ctx.filter(big, SS)[SS][0])).reshape(times, base)
    assert np.array_equal(got, np.broadcast_to(want, got.shape))
    gpu_ctx.check()

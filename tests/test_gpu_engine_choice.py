"""SneakySnake alone around the sizes where paf_filter changes its engine: one
length and threshold, offsets or thresholds per pair, and lengths per pair that
are the same, nearly the same or a mix (which above some size a sample of them
decides on the device), with a pair out of range.  A small batch is repeated on
the device; every repeat gives the small batch's results, which are compared
with the oracle's."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import pairgen
import paper_1910_03936_amd as paf
from gpu_util import assert_parity, oracle_for, results, to_device

pytestmark = pytest.mark.gpu
SS = paf.SNEAKYSNAKE
BASE = 64 * 128


def _pairs(lens, E):
    w = pairgen.Workload("choice", 0, tuple(lens), 12, 0.5, fixed_E=E, seed=pairgen.SEED_BASE + 53)
    return pairgen.generate(w, 0, BASE)


def _check(ctx, p, n, offsets, lengths, thresholds, bad=None):
    """The pairs of p over and over, n of them, with the given per-pair arrays."""
    small = to_device(p, ctx, per_pair=True, offsets=offsets)
    want = oracle_for(p, SS)
    assert_parity(results(ctx.filter(small, SS), BASE), want, "small")
    times = -(-n // BASE)
    words = small.reads.numel()
    off = None
    if offsets:
        base = torch.arange(times, device="cuda", dtype=torch.int64) * words
        off = (base[:, None] + small.word_offset[None]).reshape(-1)[:n].contiguous()
    ln = small.len.repeat(times)[:n].contiguous() if lengths else None
    E = small.E.repeat(times)[:n].contiguous() if thresholds else None
    if bad is not None:
        ln[bad] = 513
    m, e = int(p.len.max()), int(p.E.max())
    b = paf.Batch(small.reads.repeat(times), small.refs.repeat(times), n, small.stride_words, off, ln, E,
                  0 if lengths else m, 0 if thresholds else e, m, e)
    out = ctx.filter(b, SS)
    torch.cuda.synchronize()
    ids = torch.arange(n, device="cuda") % BASE
    cnt = torch.from_numpy(want[SS][1].astype(np.int32)).cuda()[ids]
    acc = torch.from_numpy(want[SS][0].astype(bool)).cuda()[ids]
    if bad is not None:
        cnt[bad], acc[bad] = 0, False
        with pytest.raises(paf.PafError):
            ctx.check()
    assert torch.equal(paf.counts_u16(out[SS][1]).to(torch.int32), cnt)
    assert torch.equal(paf.accept_bits_to_bool(out[SS][0], n), acc)
    ctx.check()


@pytest.mark.parametrize("m,E,tiles", [(250, 5, 13312), (100, 5, 16384), (250, 10, 16384), (40, 2, 14336)])
def test_one_length_and_threshold(gpu_ctx, m, E, tiles):
    p = _pairs((m,), E)
    for n in (64 * tiles, 64 * tiles + 1):
        _check(gpu_ctx, p, n, False, False, False)


@pytest.mark.parametrize("m,E,tiles", [(200, 5, 8192), (200, 9, 32768), (33, 1, 65536)])
def test_one_length(gpu_ctx, m, E, tiles):
    p = _pairs((m,), E)
    for n in (64 * tiles, 64 * tiles + 33):
        _check(gpu_ctx, p, n, True, False, False)
        _check(gpu_ctx, p, n, False, False, True)


@pytest.mark.parametrize("lens,E,tiles", [((250,), 5, 32768), ((225, 250), 10, 32768), ((64, 100, 250), 10, 32768),
                                          ((64, 150, 300), 15, 32768), ((20, 40, 64), 6, 32768), ((1, 150, 250), 2, 65536)])
def test_lengths_per_pair(gpu_ctx, lens, E, tiles):
    p = _pairs(lens, E)
    for n in (64 * tiles, 64 * tiles + 31):
        _check(gpu_ctx, p, n, True, True, False)
    _check(gpu_ctx, p, 64 * tiles + 65, False, True, True)
    _check(gpu_ctx, p, 64 * tiles + 65, True, True, True, bad=64 * tiles - 3)

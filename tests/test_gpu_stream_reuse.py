"""Streamed batches one after the other on one context: smaller and larger
ones, other stages, one and several chunks, and a call that is refused between
two that run."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import pairgen
import paper_1910_03936_amd as paf

pytestmark = pytest.mark.gpu


def _check(ctx, first, n, chunk, filters, learned=False):
    from paper_1910_03936_amd.hostbatch import host_batch
    w = pairgen.STREAM_MIX
    out, stats = paf.stream_filter(ctx, host_batch(w, n, first=first), chunk, filters, learned)
    ctx.check()
    assert stats["chunks"] == -(-n // chunk)
    p = pairgen.generate(w, first, n)
    want = oracle.filter_batch(p.reads, p.refs, p.len, p.E, filters)
    assert set(out) == set(want)
    for f, (bits, cnt) in out.items():
        assert np.array_equal(paf.accept_bits_to_bool(bits, n).numpy().astype(np.uint8), want[f][0]), (n, chunk, f)
        assert np.array_equal(paf.counts_u16(cnt).numpy(), want[f][1].astype(np.int64)), (n, chunk, f)


def test_batches_of_changing_shape(gpu_ctx):
    from paper_1910_03936_amd.hostbatch import host_batch
    gpu_ctx.mlp_set_params(pairgen.init_mlp_params())
    SS = paf.SNEAKYSNAKE
    _check(gpu_ctx, 0, 3000, 1024, SS)
    _check(gpu_ctx, 5000, 1, 64, SS)
    _check(gpu_ctx, 7000, 9001, 4096, paf.ALL_FILTERS)
    bad = host_batch(pairgen.STREAM_MIX, 5000)
    bad.len[4999] = 0
    with pytest.raises(paf.PafError):
        paf.stream_filter(gpu_ctx, bad, 1024, SS)
    bad.len[4999] = bad.max_len + 1
    with pytest.raises(paf.PafError):
        paf.stream_filter(gpu_ctx, bad, 1024, SS)
    _check(gpu_ctx, 20000, 6000, 64 * 40, SS, learned=True)
    _check(gpu_ctx, 30000, 20011, 8192, SS)
    _check(gpu_ctx, 60000, 3000, 1024, paf.GATEKEEPER)

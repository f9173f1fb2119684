"""Verification through a selection, which takes the pairs lane by lane from a
wave's list: the edges that decide where a lane reads and writes (lengths around
the words' ends up to 512, thresholds up to 31 and at or above the length), with
every pair selected; pairs out of range, selected and not; and lists longer
than 32 tiles of pairs with lengths, thresholds and offsets of their own."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import pairgen
import paper_1910_03936_amd as paf
from gpu_util import to_device

pytestmark = pytest.mark.gpu


def _dist(t):
    torch.cuda.synchronize()
    return paf.counts_u16(t).cpu().numpy().astype(np.int64)


def _bits(sel):
    words = np.zeros((sel.size + 31) // 32, np.uint32)
    at = np.nonzero(sel)[0]
    np.bitwise_or.at(words, at // 32, (np.uint32(1) << (at % 32).astype(np.uint32)))
    return torch.from_numpy(words.view(np.int32)).cuda()


def _want(p):
    return oracle.banded_batch(p.reads, p.refs, p.len, p.E).astype(np.int64)


def _edges():
    rng = np.random.default_rng(83)
    rows = []
    for m in (1, 2, 31, 32, 33, 63, 64, 65, 97, 255, 256, 257, 480, 481, 511, 512):
        a = rng.integers(0, 4, m).astype(np.uint8)
        b = a.copy()
        b[rng.integers(0, m, max(1, m // 20))] ^= 1
        tail = a.copy()
        tail[-1] ^= 2
        ins = np.concatenate([a[: m // 3], [2], a[m // 3:]])[:m].astype(np.uint8)
        for ref in (a, b, tail, ins, np.roll(a, 2), np.roll(a, -5), (a + 2) % 4, rng.integers(0, 4, m).astype(np.uint8)):
            for E in sorted({0, 1, 5, 16, min(31, m - 1), min(31, m), min(31, m + 1), 31}):
                rows.append((a, ref, m, E))
    n = len(rows)
    R, F = np.zeros((n, 512), np.uint8), np.zeros((n, 512), np.uint8)
    L, E = np.zeros(n, np.uint16), np.zeros(n, np.uint8)
    for i in rng.permutation(n):
        a, r, m, e = rows[i]
        R[i, :m], F[i, :m], L[i], E[i] = a, r, m, e
    return pairgen.Pairs(R, F, L, E, np.zeros(n, np.uint8), np.zeros(n, np.uint16))


def _some(p, ids, E=None):
    return pairgen.Pairs(p.reads[ids], p.refs[ids], p.len[ids], p.E[ids] if E is None else E, p.related[ids], p.k[ids])


@pytest.mark.parametrize("max_E", [0, 1, 5, 16, 31])
@pytest.mark.parametrize("offsets", [False, True])
def test_edges_selected(gpu_ctx, max_E, offsets):
    p = _edges()
    p = _some(p, np.nonzero(p.E <= max_E)[0])
    b = to_device(p, gpu_ctx, per_pair=True, offsets=offsets, max_len=512, max_E=max_E)
    want = _want(p)
    assert np.array_equal(_dist(gpu_ctx.verify(b, _bits(np.ones(p.n, bool)))), want)
    odd = np.arange(p.n) % 3 == 1
    got = _dist(gpu_ctx.verify(b, _bits(odd)))
    assert np.array_equal(got, np.where(odd, want, p.E.astype(np.int64) + 1))
    gpu_ctx.check()


@pytest.mark.parametrize("selected", [True, False])
@pytest.mark.parametrize("n", [500, 64 * 4096 + 100])
def test_pairs_out_of_range(gpu_ctx, selected, n):
    p = pairgen.generate(pairgen.UNEVEN_MIX, 0, n)
    b = to_device(p, gpu_ctx, per_pair=True, offsets=True, max_len=300, max_E=15)
    sel = np.arange(n) % 7 < 5
    bad = np.array([7, n // 2 + 1, n - 2])
    sel[bad] = selected
    clean = _dist(gpu_ctx.verify(b, _bits(sel)))
    gpu_ctx.check()
    ids = pairgen.sample_ids(n, min(n, 4000))
    want = np.where(sel, _want(p) if n < 1000 else 0, p.E.astype(np.int64) + 1)
    if n >= 1000:
        want[ids] = np.where(sel[ids], _want(_some(p, ids)), p.E[ids].astype(np.int64) + 1)
        assert np.array_equal(clean[ids], want[ids])
    else:
        assert np.array_equal(clean, want)
    # a threshold, a length of zero and a length above the bounds
    E, ln = b.E.clone(), b.len.clone()
    E[int(bad[0])], ln[int(bad[1])], ln[int(bad[2])] = 200, 0, 512
    broken = paf.Batch(b.reads, b.refs, n, 0, b.word_offset, ln, E, 0, 0, b.max_len, b.max_E)
    got = _dist(gpu_ctx.verify(broken, _bits(sel)))
    with pytest.raises(paf.PafError):
        gpu_ctx.check()
    assert np.all(got[bad] == 0)
    rest = np.ones(n, bool)
    rest[bad] = False
    assert np.array_equal(got[rest], clean[rest])
    gpu_ctx.check()


def test_long_lists_per_pair(gpu_ctx):
    # A small batch over and over, on lists of more than 2048 pairs (max_E 20 and up).
    base = 64 * 256
    w = pairgen.Workload("lists", 0, (40, 64, 90), 30, 0.4, e_num=31, e_den=90, seed=pairgen.SEED_BASE + 61)
    p = pairgen.generate(w, 0, base)
    b = to_device(p, gpu_ctx, per_pair=True, offsets=True)
    assert b.max_E >= 20
    want = _want(p)
    times = 400
    words = b.reads.numel()
    off = (torch.arange(times, device="cuda", dtype=torch.int64)[:, None] * words + b.word_offset[None]).reshape(-1).contiguous()
    big = paf.Batch(b.reads.repeat(times), b.refs.repeat(times), base * times, 0, off, b.len.repeat(times),
                    b.E.repeat(times), 0, 0, b.max_len, b.max_E)
    sel = np.random.default_rng(5).random(base) < 0.3
    got = _dist(gpu_ctx.verify(big, _bits(sel).repeat(times))).reshape(times, base)
    assert np.array_equal(got, np.broadcast_to(np.where(sel, want, p.E.astype(np.int64) + 1), got.shape))
    gpu_ctx.check()

"""MAGNET where its launches change form: the pairs that a group of lanes takes
together (16, 32 or 64 lanes a pair: thresholds 7 and 8, 15 and 16), when every
pair of a tile is one or a few are; and batches with max_E 0, whose pairs are
only compared, at lengths around the words' ends.  Whole numbers: they equal
the oracle's."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import pairgen
import paper_1910_03936_amd as paf
from gpu_util import assert_parity, results, to_device

pytestmark = pytest.mark.gpu


def _check(ctx, reads, refs, ln, E, per_pair, label):
    n = len(ln)
    p = pairgen.Pairs(reads, refs, ln.astype(np.int32), np.broadcast_to(E, n).astype(np.int32), np.ones(n, bool),
                      np.zeros(n, np.int32))
    got = results(ctx.filter_magnet(to_device(p, ctx, per_pair=per_pair, offsets=per_pair)), n)
    assert_parity(got, {paf.SNEAKYSNAKE: oracle.magnet_batch(p.reads, p.refs, p.len, p.E)}, label)
    ctx.check()


@pytest.mark.parametrize("E", [7, 8, 15, 16])
@pytest.mark.parametrize("share", [1.0, 0.05])
def test_pairs_taken_by_groups(gpu_ctx, E, share):
    # Homopolymers with an edit or two: long runs on every diagonal.
    rng = np.random.default_rng(E)
    lens = np.array([64, 250, 512])[rng.integers(0, 3, 64 * 5 + 3)]
    n, M = lens.size, 512
    reads, refs = np.zeros((n, M), np.uint8), np.zeros((n, M), np.uint8)
    for i, m in enumerate(lens):
        a = np.full(m, rng.integers(0, 4), np.uint8) if rng.random() < share else rng.integers(0, 4, m).astype(np.uint8)
        b = a.copy()
        for x in (a, b):
            at = rng.integers(0, m, rng.integers(0, 3))
            x[at] = (x[at] + 1) % 4
        reads[i, :m], refs[i, :m] = a, b
    _check(gpu_ctx, reads, refs, lens, E, True, f"E={E} share={share}")
    same = lens == 250
    _check(gpu_ctx, reads[same][:, :250].copy(), refs[same][:, :250].copy(), lens[same], E, False, f"uniform E={E} share={share}")


@pytest.mark.parametrize("lens", [(1,), (32,), (33, 64, 65), (250, 256, 257), (511, 512), (1, 31, 63, 512)])
def test_equal_pairs_only(gpu_ctx, lens):
    # Every position of a single edit, no edit, and unrelated pairs.
    rng = np.random.default_rng(sum(lens))
    rows = []
    for m in lens:
        a = rng.integers(0, 4, m).astype(np.uint8)
        for at in [None, *range(0, m, max(1, m // 40)), m - 1]:
            b = a.copy()
            if at is not None:
                b[at] ^= 1 + at % 3
            rows.append((a, b, m))
        rows.append((a, rng.integers(0, 4, m).astype(np.uint8), m))
    rows = [rows[i] for i in rng.permutation(len(rows))]
    n, M = len(rows), max(lens)
    reads, refs = np.zeros((n, M), np.uint8), np.zeros((n, M), np.uint8)
    for i, (a, b, m) in enumerate(rows):
        reads[i, :m], refs[i, :m] = a, b
    ln = np.array([m for _, _, m in rows])
    _check(gpu_ctx, reads, refs, ln, 0, True, f"lens={lens}")
    if len(lens) == 1:
        _check(gpu_ctx, reads, refs, ln, 0, False, f"uniform {lens}")


def _repeated(ctx, p, n):
    """p's pairs over and over, n of them: every repeat gives p's counts and decisions."""
    b = to_device(p, ctx, per_pair=False, offsets=False)
    acc, cnt = oracle.magnet_batch(p.reads, p.refs, p.len, p.E)
    times = -(-n // p.n)
    big = paf.Batch(b.reads.repeat(times), b.refs.repeat(times), n, b.stride_words, uniform_len=b.uniform_len,
                    uniform_E=b.uniform_E, max_len=b.max_len, max_E=b.max_E)
    out = ctx.filter_magnet(big)[paf.SNEAKYSNAKE]
    ids = torch.arange(n, device="cuda") % p.n
    assert torch.equal(paf.counts_u16(out[1]).to(torch.int32), torch.from_numpy(cnt.astype(np.int32)).cuda()[ids])
    assert torch.equal(paf.accept_bits_to_bool(out[0], n), torch.from_numpy(acc.astype(bool)).cuda()[ids])
    ctx.check()


@pytest.mark.parametrize("m,n", [(20, 64 * 8 * 5 + 3), (64, 64 * 4 * 9 + 33), (100, 64 * 3), (150, 64 * 7 + 1), (512, 321)])
def test_equal_pairs_over_several_tiles(gpu_ctx, m, n):
    w = pairgen.Workload("equal", 0, (m,), 1, 0.3, fixed_E=0, seed=pairgen.SEED_BASE + 67)
    _repeated(gpu_ctx, pairgen.generate(w, 0, 1999), n)


@pytest.mark.parametrize("E", [1, 3, 4])
def test_pairs_without_an_obstacle(gpu_ctx, E):
    # Lists of more tiles than counts are loaded at a time, half of the pairs equal.
    w = pairgen.Workload("free", 0, (100,), 1, 0.2, fixed_E=E, seed=pairgen.SEED_BASE + 71)
    _repeated(gpu_ctx, pairgen.generate(w, 0, 64 * 63 + 5), 64 * 2048 * 17 + 77)

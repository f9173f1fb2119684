"""Narrow sub-mazes (walked all at once) on both sides of the rule that picks
them, with and without a cap, at thresholds of every register class, and the
chunk sizes that a batch's size picks, against the oracle: whole numbers."""
from __future__ import annotations

import pytest

import oracle
import pairgen
import paper_1910_03936_amd as paf
from gpu_util import assert_parity, results, to_device

pytestmark = pytest.mark.gpu
SS = paf.SNEAKYSNAKE


@pytest.mark.parametrize("E", [1, 4, 8, 12, 20, 31])
def test_widths_and_caps(gpu_ctx, E):
    p = pairgen.generate(pairgen.FIXED_250BP.with_E(E), 401 + E, 64 * 9 + 5)
    b = to_device(p, gpu_ctx, per_pair=False, offsets=False)
    for t in (2, 3, 4, 7, 11, 15, 16, 17):
        a, c = oracle.sneakysnake_t_batch(p.reads, p.refs, p.len, p.E, t)
        assert_parity(results(gpu_ctx.filter_partitioned(b, t), p.n), {SS: (a, c)}, f"E={E} t={t}")
        for y in (1, 2, 5):
            a, c = oracle.sneakysnake_fpga_batch(p.reads, p.refs, p.len, p.E, t, y)
            assert_parity(results(gpu_ctx.filter_partitioned(b, t, y), p.n), {SS: (a, c)}, f"E={E} t={t} y={y}")
    gpu_ctx.check()


@pytest.mark.parametrize("per_pair", [False, True])
def test_chunk_sizes(gpu_ctx, per_pair):
    tiles = 8 * 256
    for n in (1, 64 * tiles, 64 * 2 * tiles - 1, 64 * 2 * tiles + 1, 64 * 5 * tiles + 77):
        w = pairgen.SMALL_100BP if not per_pair else pairgen.UNEVEN_MIX
        p = pairgen.generate(w, 0, n)
        b = to_device(p, gpu_ctx, per_pair=per_pair, offsets=per_pair)
        a, c = oracle.sneakysnake_t_batch(p.reads, p.refs, p.len, p.E, 8)
        assert_parity(results(gpu_ctx.filter_partitioned(b, 8), n), {SS: (a, c)}, f"n={n}")
    gpu_ctx.check()


@pytest.mark.parametrize("E", [15, 16, 31])
def test_widest_narrow_form(gpu_ctx, E):
    # One replication: the form changes after 12 columns from the class of 20 on.
    for per_pair in (False, True):
        w = pairgen.UNEVEN_MIX if per_pair else pairgen.FIXED_250BP.with_E(E)
        p = pairgen.generate(w, 77, 64 * 7 + 9)
        b = to_device(p, gpu_ctx, per_pair=per_pair, offsets=per_pair, max_E=E)
        for t in (12, 13, 16, 17):
            a, c = oracle.sneakysnake_fpga_batch(p.reads, p.refs, p.len, p.E, t, 1)
            assert_parity(results(gpu_ctx.filter_partitioned(b, t, 1), p.n), {SS: (a, c)}, f"E={E} t={t} {per_pair}")
    gpu_ctx.check()

"""SneakySnake of per-pair and small batches (each lane's window at its own
column) against the oracle: lengths and thresholds at the edges of words and
threshold classes, batch sizes around a tile, and a batch whose waves take more
pairs than their ring of counts holds."""
from __future__ import annotations

import pytest

import pairgen
import paper_1910_03936_amd as paf
from gpu_util import assert_parity, oracle_for, results, to_device

pytestmark = pytest.mark.gpu
SS = paf.SNEAKYSNAKE


def _w(lens, E, kmax=12, unrelated=0.4):
    return pairgen.Workload("flow", 0, tuple(lens), kmax, unrelated, fixed_E=E, seed=pairgen.SEED_BASE + 41)


@pytest.mark.parametrize("m,E", [(1, 0), (5, 7), (31, 3), (32, 9), (33, 31), (64, 4), (65, 11), (95, 1), (96, 13),
                                 (150, 6), (250, 9), (250, 16), (257, 21), (511, 26), (512, 31)])
def test_edges_of_words_and_classes(gpu_ctx, m, E):
    for n in (1, 63, 64, 65, 2500):
        p = pairgen.generate(_w((m,), E), 3, n)
        want = oracle_for(p, SS)
        b = to_device(p, gpu_ctx, per_pair=False, offsets=False)
        assert_parity(results(gpu_ctx.filter(b, SS), n), want, f"m={m} E={E} n={n}")
        # the same pairs under wider bounds and with per-pair arrays
        b = to_device(p, gpu_ctx, per_pair=False, offsets=False, max_len=min(512, m + 70), max_E=min(31, E + 9))
        assert_parity(results(gpu_ctx.filter(b, SS), n), want, f"m={m} E={E} n={n} wider bounds")
        b = to_device(p, gpu_ctx, per_pair=True, offsets=True)
        assert_parity(results(gpu_ctx.filter(b, SS), n), want, f"m={m} E={E} n={n} per pair")
    gpu_ctx.check()


def test_more_pairs_than_the_ring_holds(gpu_ctx):
    n = 64 * 4096 * 18 + 17
    p = pairgen.generate(_w((20, 40, 64), 3), 0, n)
    b = to_device(p, gpu_ctx, per_pair=True, offsets=True)
    assert_parity(results(gpu_ctx.filter(b, SS), n), oracle_for(p, SS), "ring")
    gpu_ctx.check()

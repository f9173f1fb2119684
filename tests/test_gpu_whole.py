"""GateKeeper and Shouji (alone, together and with SneakySnake) against the
oracle at the edges of words, windows and threshold classes: runs of free cells
that touch a pair's ends, windows with and without vacant cells, thresholds
inside a class, and an odd and an even number of windows."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import pairgen
import paper_1910_03936_amd as paf
from gpu_util import assert_parity, oracle_for, results, to_device

pytestmark = pytest.mark.gpu
SS, GK, SH = paf.SNEAKYSNAKE, paf.GATEKEEPER, paf.SHOUJI


@pytest.mark.parametrize("m,E", [(1, 0), (1, 2), (2, 1), (3, 3), (4, 31), (31, 2), (32, 3), (33, 8), (34, 1), (63, 4),
                                 (64, 9), (66, 10), (97, 6), (128, 11), (160, 0), (250, 5), (250, 13), (257, 20),
                                 (300, 16), (511, 25), (512, 31)])
def test_masks_at_edges(gpu_ctx, m, E):
    n = 333
    w = pairgen.Workload("whole", 0, (m,), max(2, m // 8), 0.4, fixed_E=E, seed=pairgen.SEED_BASE + 43)
    p = pairgen.generate(w, 1, n)
    # some pairs without edits, shifted by up to E, or differing at an end only
    for i in range(0, 60, 3):
        p.refs[i, :m] = p.reads[i, :m]
        p.refs[i + 1, :m] = np.roll(p.reads[i + 1, :m], (i // 3) % (E + 1))
        p.refs[i + 2, :m] = p.reads[i + 2, :m]
        p.refs[i + 2, [0, m - 1, min(m - 1, 1 + i % 4)]] ^= 1
    want = oracle_for(p, paf.ALL_FILTERS)
    uniform = to_device(p, gpu_ctx, per_pair=False, offsets=False)
    wider = to_device(p, gpu_ctx, per_pair=False, offsets=False, max_len=min(512, m + 33), max_E=min(31, E + 4))
    pairs = to_device(p, gpu_ctx, per_pair=True, offsets=True)
    for f in (GK, SH, GK | SH, SS | GK, SS | SH, paf.ALL_FILTERS):
        sel = {k: want[k] for k in want if k & f}
        for tag, b in (("uniform", uniform), ("wider", wider), ("per pair", pairs)):
            assert_parity(results(gpu_ctx.filter(b, f), n), sel, f"m={m} E={E} mask={f} {tag}")
        assert_parity(results(gpu_ctx.filter_persistent(uniform, f), n), sel, f"m={m} E={E} mask={f} persistent")
    gpu_ctx.check()


def test_lengths_and_thresholds_mixed_in_a_wave(gpu_ctx):
    rng = np.random.default_rng(5)
    n, cs = 4000, 300
    p = pairgen.generate(pairgen.UNEVEN_MIX, 9, n, stride=cs)
    p.len[:] = rng.integers(1, cs + 1, n)
    p.E[:] = rng.integers(0, 32, n)
    b = to_device(p, gpu_ctx, per_pair=True, offsets=True)
    for f in (GK, SH, paf.ALL_FILTERS):
        want = oracle_for(p, f)
        assert_parity(results(gpu_ctx.filter(b, f), n), want, f"mask={f}")
        o = torch.randperm(n, generator=torch.Generator().manual_seed(f)).to(torch.int32).cuda()
        assert_parity(results(gpu_ctx.filter_ordered(b, o, f), n), want, f"mask={f} ordered")
    gpu_ctx.check()

"""GPU encoder against the host encoder: lengths around a word, rows that start
at any byte, spare bytes after a row that hold anything, and codes above 3."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import paper_1910_03936_amd as paf

pytestmark = pytest.mark.gpu


def _host(codes, lens, m, off, stride, total):
    lib = paf.load_library()
    words = np.zeros(total, np.uint64)
    p = lambda a: None if a is None else a.ctypes.data_as(ctypes.c_void_p)
    assert lib.paf_pack_host(p(codes), codes.shape[1], p(lens), m, p(off), stride, codes.shape[0], p(words), 4) == 0
    return words


@pytest.mark.parametrize("m", [1, 3, 31, 32, 33, 63, 64, 100, 250, 251, 511, 512])
@pytest.mark.parametrize("spare,shift", [(0, 0), (1, 1), (7, 3)])
def test_uniform_rows(gpu_ctx, m, spare, shift):
    rng = np.random.default_rng(m * 10 + spare)
    for n in (1, 2, 257):
        codes = rng.integers(0, 4, (n, m + spare), dtype=np.uint8)
        codes[:, m:] = 0xFF                       # bytes past a sequence are not looked at
        buf = torch.zeros(codes.size + shift, dtype=torch.uint8, device="cuda")
        dev = buf[shift:].view(n, m + spare)
        dev.copy_(torch.from_numpy(codes))
        for stride in (paf.words_for(m), paf.words_for(m) + 2):
            got = gpu_ctx.pack(dev, uniform_len=m, stride_words=stride).cpu().numpy().view(np.uint64)
            assert np.array_equal(got, _host(codes, None, m, None, stride, n * stride)), (n, stride)
    gpu_ctx.check()


def test_per_row_lengths_and_bad_codes(gpu_ctx):
    rng = np.random.default_rng(3)
    n, cs = 1000, 301
    codes = rng.integers(0, 4, (n, cs), dtype=np.uint8)
    lens = rng.integers(1, cs + 1, n).astype(np.uint16)
    w = (lens.astype(np.int64) + 31) // 32
    off = np.concatenate([[0], np.cumsum(w)[:-1]]).astype(np.uint64)
    dev = torch.from_numpy(codes).cuda()
    ln = torch.from_numpy(lens.astype(np.int16)).cuda()
    of = torch.from_numpy(off.astype(np.int64)).cuda()
    got = gpu_ctx.pack(dev, ln, word_offset=of, total_words=int(w.sum())).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, _host(codes, lens, 0, off, 0, int(w.sum())))
    gpu_ctx.check()
    for value in (4, 0x80):
        dev[n - 1, int(lens[n - 1]) - 1] = value
        gpu_ctx.pack(dev, ln, word_offset=of, total_words=int(w.sum()))
        with pytest.raises(paf.PafError):
            gpu_ctx.check()
        gpu_ctx.check()

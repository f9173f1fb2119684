"""The work that performance figures of this library are quoted on.

Each case is one call (or one training step) through the public entry points
of paper_1910_03936_amd, on synthetic pairs with the shapes of the thesis's
evaluation sets: a read of i.i.d. bases, and a reference segment that is
either unrelated or the read with up to `kmax` edits.  Pairs are made on the
GPU from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1910_03936_amd as paf

SS, GK, SH = paf.SNEAKYSNAKE, paf.GATEKEEPER, paf.SHOUJI
UNEVEN_LENS = (64, 100, 150, 250, 300)   # read lengths of the uneven mix
STREAM_LENS = (100, 150, 250)            # read lengths of the streamed mix
LEARN_ROWS = 65536                       # pairs the cost model of a learned case is trained on

# What a case may hold:
#   op         the entry point
#   pairs      pairs (training: rows) of one call
#   length     bases per sequence of a uniform batch, or 0 for a mix
#   lens       "uneven" or "stream": per-pair lengths of that mix
#   E          threshold, or -1 for floor(e_pct m / 100) per pair
#   filters    mask of decision stages
#   t, y       sub-maze width and obstacle cap of the partitioned filter
#   unrelated  percent of the pairs with an unrelated segment; kmax: most edits of a related one


def _pairs(op, name, pairs, length=0, E=-1, **more):
    c = {"name": name, "op": op, "pairs": pairs, "length": length, "E": E, "unrelated": 70, "kmax": 40}
    c.update(more)
    return c


def listed():
    return [
        # The seeds of a single read, or a serving request: latency counts.
        _pairs("filter", "filter-1k-100bp-E5", 1000, 100, 5, filters=SS, unrelated=50, kmax=15),
        # The small evaluation set: one short batch of 100 bp pairs.
        _pairs("filter", "filter-100k-100bp-E5", 100_000, 100, 5, filters=SS, unrelated=50, kmax=15),
        # The headline batch: 250 bp candidates of a mapper, resident on the GPU.
        _pairs("filter", "filter-10M-250bp-E10", 10_000_000, 250, 10, filters=SS),
        # Reads of several sequencers in one batch: lengths, thresholds and offsets per pair.
        _pairs("filter", "filter-2M-uneven", 2_000_000, lens="uneven", e_pct=5, filters=SS),
        # The three decision stages side by side, as their accuracy is compared.
        _pairs("filter", "stages-2M-250bp-E10", 2_000_000, 250, 10, filters=SS | GK | SH),
        # SneakySnake-5: the maze cut into sub-mazes of five columns.
        _pairs("partitioned", "partitioned-2M-250bp-t5", 2_000_000, 250, 10, t=5, y=0),
        # MAGNET, the most accurate and the slowest stage.
        _pairs("magnet", "magnet-1M-250bp-E10", 1_000_000, 250, 10),
        # Banded edit distance of the pairs SneakySnake accepted.
        _pairs("verify", "verify-4M-250bp-E10", 4_000_000, 250, 10),
        # The encoder: base codes of a batch's reads and segments into packed words.
        _pairs("encode", "encode-1M-250bp", 1_000_000, 250, 10),
        # The learned pipeline: cost levels from the model, then the filter in their order.
        _pairs("learned", "learned-4M-250bp-E10", 4_000_000, 250, 10),
        # One minibatch of the cost model's training: loss, gradients and Adam's update.
        {"name": "train-4096", "op": "train", "pairs": 4096},
        # Pairs in pinned host memory, copied and filtered chunk by chunk.
        _pairs("stream", "stream-2M-mix", 2_000_000, lens="stream", e_pct=10, filters=SS, unrelated=80, chunk=524_288),
    ]


# Cost of a pair of each kind of call next to SneakySnake's whole-maze filter,
# so that a drawn case costs no more than the largest listed one.
_WEIGHT = {"filter": 1.0, "partitioned": 2.0, "magnet": 12.0, "verify": 3.0, "encode": 8.0, "learned": 2.5,
           "stream": 4.0}


def draw(rng):
    op = rng.choice(["filter"] * 4 + ["partitioned", "magnet", "verify", "encode", "learned", "train", "stream"])
    if op == "train":
        return {"op": "train", "pairs": int(round(math.exp(rng.uniform(math.log(256), math.log(32768)))))}
    c = {"op": op, "unrelated": rng.choice([50, 70, 80]), "kmax": rng.choice([15, 40])}
    if op == "stream" or (op in ("filter", "verify", "partitioned", "magnet") and rng.random() < 0.3):
        c.update(length=0, E=-1, lens=rng.choice(["uneven", "stream"]), e_pct=rng.choice([2, 5, 10]))
        m, E = 300, 30 * c["e_pct"] // 10
    else:
        m = rng.choice([100, 150, 250, rng.randint(50, 500)])
        E = rng.randint(0, min(31, m // 10))
        c.update(length=m, E=E)
    weight = _WEIGHT[op]
    if op in ("filter", "stream"):
        # SneakySnake alone is what a mapper runs; the others are run for comparison.
        c["filters"] = SS if op == "stream" else rng.choice([SS, SS, GK, SH, GK | SH, SS | GK | SH])
        weight *= 8.0 if c["filters"] != SS else 1.0
    if op == "partitioned":
        c["t"], c["y"] = rng.choice([(5, 0), (10, 0), (25, 0), (50, 0), (8, 3)])
    grow = max(1.0, (2 * E + 1) / 21.0)
    weight *= grow * grow if op == "magnet" else grow
    most = 10_000_000 * 8 / (paf.words_for(m) * weight)
    least = 100_000 if op == "stream" else 100
    c["pairs"] = int(math.exp(rng.uniform(math.log(least), math.log(max(2 * least, most)))))
    if op == "stream":
        c["chunk"] = max(64, (c["pairs"] // 4) // 64 * 64)
    return c


# -- inputs -------------------------------------------------------------------

def _lens_E(case, gen, dev):
    """Per-pair lengths and thresholds (int32), from the case's mix."""
    n = case["pairs"]
    if case.get("lens"):
        mix = torch.tensor(UNEVEN_LENS if case["lens"] == "uneven" else STREAM_LENS, dtype=torch.int32, device=dev)
        ln = mix[torch.randint(0, mix.numel(), (n,), generator=gen, device=dev)]
        return ln, ln * case["e_pct"] // 100
    return (torch.full((n,), case["length"], dtype=torch.int32, device=dev),
            torch.full((n,), case["E"], dtype=torch.int32, device=dev))


def _codes(case, ln, m, gen, dev):
    """(reads, refs) uint8 codes [len(ln), m] of one slice of the batch."""
    n = ln.shape[0]
    r = torch.randint(0, 1 << 31, (n, m), generator=gen, device=dev, dtype=torch.int32)
    row = torch.randint(0, 1 << 31, (n, 2), generator=gen, device=dev, dtype=torch.int32)
    reads = ((r >> 26) & 3).to(torch.uint8)
    # k ~ U{0..kmax} edits spread evenly over the read, a third of each kind.
    k = row[:, 0] % (case["kmax"] + 1)
    edit = (r & 0xFFFF) < (k * 65536 // ln)[:, None]
    kind = ((r >> 16) & 0xFF) % 3                      # substitution, insertion, deletion
    step = torch.where(edit & (kind == 2), 1, torch.where(edit & (kind == 1), -1, 0)).to(torch.int8)
    src = torch.cumsum(step, 1, dtype=torch.int16).to(torch.int64)
    del step
    src += torch.arange(m, device=dev)
    base = ((r >> 24) & 3).to(torch.uint8)             # random bases of the segment
    outside = (src < 0) | (src >= m) | (edit & (kind == 1)) | ((row[:, 1] % 100) < case["unrelated"])[:, None]
    refs = torch.gather(reads, 1, src.clamp_(0, m - 1))
    sub = edit & (kind == 0)
    refs = torch.where(sub, (refs + 1 + base % 3) & 3, refs)
    return reads, torch.where(outside, base, refs)


def _batch(case, ctx, seed):
    """The case's pairs, packed and resident on the GPU."""
    dev = torch.device("cuda", ctx.device)
    gen = torch.Generator(device=dev).manual_seed(seed)
    ln, E = _lens_E(case, gen, dev)
    n = case["pairs"]
    mixed = bool(case.get("lens"))
    m = max(UNEVEN_LENS if case["lens"] == "uneven" else STREAM_LENS) if mixed else case["length"]
    rows = max(1, (1 << 25) // m)
    rd, rf = [], []
    for a in range(0, n, rows):
        l = ln[a:a + rows]
        reads, refs = _codes(case, l, m, gen, dev)
        if mixed:
            w = (l.to(torch.int64) + 31) // 32
            end = torch.cumsum(w, 0)
            l16, total = l.to(torch.int16), int(end[-1])
            rd.append(ctx.pack(reads, l16, word_offset=end - w, total_words=total))
            rf.append(ctx.pack(refs, l16, word_offset=end - w, total_words=total))
        else:
            rd.append(ctx.pack(reads, uniform_len=m))
            rf.append(ctx.pack(refs, uniform_len=m))
        del reads, refs
    rd, rf = torch.cat(rd), torch.cat(rf)
    if mixed:
        w = (ln.to(torch.int64) + 31) // 32
        off = torch.cumsum(w, 0) - w
        return paf.Batch(rd, rf, n, 0, off, ln.to(torch.int16), E.to(torch.uint8), max_len=int(ln.max()),
                         max_E=int(E.max()))
    return paf.Batch(rd, rf, n, paf.words_for(m), uniform_len=m, uniform_E=case["E"], max_len=m, max_E=case["E"])


def _init_params(rng):
    """He-uniform weights and zero biases of the 64 -> 128 -> 128 -> 1 cost model."""
    parts = []
    for rows, fan_in in ((128, 64), (128, 128), (1, 128)):
        a = math.sqrt(6.0 / fan_in)
        parts += [rng.uniform(-a, a, rows * fan_in), np.zeros(rows)]
    return np.concatenate(parts).astype(np.float32)


TRAIN_MIX = {"lens": "uneven", "e_pct": 5, "length": 0, "E": -1, "unrelated": 70, "kmax": 40}


def _rows(ctx, pairs, seed):
    """Training rows of the uneven mix: features, and SneakySnake's counts at E = 31."""
    b = _batch(dict(TRAIN_MIX, pairs=pairs), ctx, seed)
    lab = ctx.filter(paf.Batch(b.reads, b.refs, pairs, 0, b.word_offset, b.len, None, 0, 31, b.max_len, 31), SS)
    return ctx.features(b), lab[SS][1]


def _train_inputs(case, seed):
    """A minibatch of the uneven mix in plain torch: the 64 features of each pair (m / 512, E / 32, and the
    share of matching cells in the first 64 columns of each diagonal within E), a target like SneakySnake's
    count (the mismatches of a pair's start, or one obstacle in five columns; at most 32), and the model's
    first weights."""
    dev = torch.device("cuda", 0)
    gen = torch.Generator(device=dev).manual_seed(seed)
    c = dict(TRAIN_MIX, pairs=case["pairs"])
    n, m = c["pairs"], max(UNEVEN_LENS)
    ln, E = _lens_E(c, gen, dev)
    reads, refs = _codes(c, ln, m, gen, dev)
    feats = torch.zeros((n, 64), dtype=torch.float32, device=dev)
    feats[:, 0], feats[:, 1] = ln / 512, E / 32
    col = torch.arange(64, device=dev)
    for d in range(-15, 16):
        at = col + d
        same = (reads[:, at.clamp(0, m - 1)] == refs[:, :64]) & (at >= 0) & (at[None] < ln[:, None])
        feats[:, 32 + d] = torch.where(E >= abs(d), same.sum(1) / 64, 0.0)
    off = (reads[:, :64] != refs[:, :64]).sum(1)
    targets = torch.where(off < 40, off, ln // 5).clamp(max=32).to(torch.float32)
    return feats, targets, _init_params(np.random.default_rng(seed))


def prepare(case, seed):
    ctx = paf.Context(0)
    dev = torch.device("cuda", 0)
    op = case["op"]
    if op == "train":
        feats, targets, params = _train_inputs(case, seed)
        ctx.mlp_set_params(params)
        return {"op": op, "ctx": ctx, "feats": feats, "targets": targets}
    if op == "encode":
        gen = torch.Generator(device=dev).manual_seed(seed)
        reads, refs = _encode_codes(case, gen, dev)
        return {"op": op, "ctx": ctx, "reads": reads, "refs": refs, "m": case["length"], "E": case["E"]}
    b = _batch(case, ctx, seed)
    s = {"op": op, "ctx": ctx, "batch": b}
    n = b.n_pairs
    if op == "filter":
        s["filters"] = case["filters"]
        s["out"] = ctx.alloc_out(n, case["filters"], dev)
    elif op == "partitioned":
        s.update(t=case["t"], y=case["y"], out=ctx.alloc_out(n, SS, dev))
    elif op == "magnet":
        s["out"] = ctx.alloc_out(n, SS, dev)
    elif op == "verify":
        s["select"] = ctx.filter(b, SS)[SS][0]
        s["dist"] = torch.empty(n, dtype=torch.int16, device=dev)
    elif op == "learned":
        feats, labels = _rows(ctx, LEARN_ROWS, seed + 1_000_003)
        ctx.mlp_set_params(_init_params(np.random.default_rng(seed)))
        ctx.mlp_train(feats, labels, 2, 2048, 1e-3)
        s["out"] = ctx.alloc_out(n, SS, dev)
    elif op == "stream":
        def pin(t):
            h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
            return h.copy_(t)
        hb = paf.HostBatch(pin(b.reads), pin(b.refs), pin(b.len), pin(b.E), b.max_len, b.max_E)
        out = {SS: (torch.zeros((n + 31) // 32, dtype=torch.int32, pin_memory=True),
                    torch.zeros(n, dtype=torch.int16, pin_memory=True))}
        s = {"op": op, "ctx": ctx, "host": hb, "out": out, "filters": case["filters"], "chunk": case["chunk"]}
    return s


def _encode_codes(case, gen, dev):
    n, m = case["pairs"], case["length"]
    ln, _ = _lens_E(case, gen, dev)
    rows = max(1, (1 << 25) // m)
    got = [_codes(case, ln[a:a + rows], m, gen, dev) for a in range(0, n, rows)]
    return torch.cat([r for r, _ in got]), torch.cat([f for _, f in got])


# -- one pass -----------------------------------------------------------------

def run(s):
    ctx, op = s["ctx"], s["op"]
    if op == "filter":
        return ctx.filter(s["batch"], s["filters"], out=s["out"])
    if op == "partitioned":
        return ctx.filter_partitioned(s["batch"], s["t"], s["y"], out=s["out"])
    if op == "magnet":
        return ctx.filter_magnet(s["batch"], out=s["out"])
    if op == "verify":
        return ctx.verify(s["batch"], s["select"], dist=s["dist"])
    if op == "encode":
        b = ctx.pack_pairs(s["reads"], s["refs"], uniform_len=s["m"], uniform_E=s["E"])
        return b.reads, b.refs
    if op == "learned":
        return ctx.filter_bucketed_local(s["batch"], out=s["out"])
    if op == "train":
        loss, grads = ctx.mlp_train_step(s["feats"], s["targets"], 1e-3, want_grads=True)
        return {"loss": loss, "grads": grads}
    if op == "stream":
        out, _ = paf.stream_filter(ctx, s["host"], s["chunk"], s["filters"], out=s["out"])
        return out
    raise ValueError(op)


# -- what a pass cannot do without --------------------------------------------

def _mean_words(case):
    if not case.get("lens"):
        return float(paf.words_for(case["length"]))
    mix = UNEVEN_LENS if case["lens"] == "uneven" else STREAM_LENS
    return sum(paf.words_for(m) for m in mix) / len(mix)


def work(case):
    n = case["pairs"]
    if case["op"] == "train":
        params = paf.MLP_NPARAMS
        macs = 64 * 128 + 128 * 128 + 128
        # Rows and targets in; weights and moments in and out; gradients out.
        # Forward, and both products of the backward pass (none for the inputs' gradient).
        return {"bytes": n * (64 * 4 + 4) + 7 * 4 * params, "flops": 2 * n * (3 * macs - 64 * 128)}
    words = 16.0 * _mean_words(case)                       # both sequences of a pair
    per_pair = 11 if case.get("lens") and case["op"] != "stream" else (3 if case.get("lens") else 0)
    if case["op"] == "encode":
        return {"bytes": n * (2.0 * case["length"] + words), "flops": 0}
    if case["op"] == "verify":
        # Selection bits in, a distance out for every pair; sequences of the selected pairs
        # only, which are a tenth of a batch or more.
        return {"bytes": n * (0.125 + 2.0 + 0.1 * (words + per_pair)), "flops": 0}
    stages = bin(case.get("filters", SS)).count("1")
    return {"bytes": n * (words + per_pair + stages * 2.125), "flops": 0}


def exact(case, seed):
    """The training step's loss and gradients in 64 bits; every other case returns whole numbers."""
    if case["op"] != "train":
        return None
    feats, targets, params = _train_inputs(case, seed)
    X, t = feats.double(), targets.double()
    p = torch.from_numpy(params.astype(np.float64)).to(X.device)
    W1, b1, W2, b2, W3, b3 = torch.split(p, [8192, 128, 16384, 128, 128, 1])
    W1, W2 = W1.view(128, 64), W2.view(128, 128)
    h1 = (X @ W1.T + b1).clamp_min(0)
    h2 = (h1 @ W2.T + b2).clamp_min(0)
    e = h2 @ W3 + b3 - t
    dy = 2.0 * e / X.shape[0]
    d2 = dy[:, None] * W3 * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    grads = torch.cat([(d1.T @ X).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), h2.T @ dy,
                       dy.sum().reshape(1)])
    return {"loss": (e * e).mean().reshape(1), "grads": grads}

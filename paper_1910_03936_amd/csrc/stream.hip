// Streaming filter: pairs held in host memory are copied chunk by chunk to
// the device on a copy stream while the previous chunk is filtered on a
// compute stream (double-buffered), the way the FPGA system streamed pairs
// over PCIe and returned one decision bit per pair (Ch. 4, Secs. 4.2-4.4).
#include <string.h>

#include <algorithm>
#include <chrono>
#include <new>
#include <thread>
#include <vector>

#include "paf_internal.h"

using namespace paf;

namespace {

// Word offsets of a chunk's pairs from their lengths: an exclusive scan of
// ceil(len / 32) in three passes (block sums, scan of the sums, apply).
constexpr int kScanBlock = 1024;

__global__ void __launch_bounds__(256) words_block_sum_kernel(const uint16_t* len, uint64_t n, uint32_t* sums) {
    __shared__ uint32_t red[256];
    const uint64_t base = (uint64_t)blockIdx.x * kScanBlock;
    uint32_t s = 0;
    for (uint32_t i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        const uint64_t p = base + i;
        if (p < n) s += (len[p] + 31u) >> 5;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (uint32_t o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = red[0];
}

// One block: exclusive scan of the block sums into 64-bit bases.
__global__ void __launch_bounds__(1024) block_base_kernel(const uint32_t* sums, uint32_t nb, uint64_t* base) {
    __shared__ uint64_t wtot[16];
    __shared__ uint64_t carry;
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t == 0) carry = 0;
    __syncthreads();
    for (uint32_t b0 = 0; b0 < nb; b0 += 1024) {
        const uint64_t v = b0 + t < nb ? sums[b0 + t] : 0u;
        uint64_t inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t o = __shfl_up(inc, off);
            if (lane >= (uint32_t)off) inc += o;
        }
        if (lane == 63) wtot[wv] = inc;
        __syncthreads();
        uint64_t before = carry;
        for (uint32_t w = 0; w < wv; ++w) before += wtot[w];
        if (b0 + t < nb) base[b0 + t] = before + inc - v;
        __syncthreads();
        if (t == 0) {
            uint64_t tot = 0;
            for (int w = 0; w < 16; ++w) tot += wtot[w];
            carry += tot;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kScanBlock) words_offset_kernel(const uint16_t* len, uint64_t n,
                                                                   const uint64_t* base, uint64_t* off) {
    __shared__ uint32_t wtot[16];
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const uint64_t p = (uint64_t)blockIdx.x * kScanBlock + t;
    const uint32_t v = p < n ? ((len[p] + 31u) >> 5) : 0u;
    uint32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc, o);
        if (lane >= (uint32_t)o) inc += x;
    }
    if (lane == 63) wtot[wv] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wv; ++w) before += wtot[w];
    if (p < n) off[p] = base[blockIdx.x] + before + inc - v;
}

struct Slot {
    uint64_t* rd = nullptr;
    uint64_t* rf = nullptr;
    uint16_t* len = nullptr;
    uint8_t* E = nullptr;
    uint64_t* off = nullptr;
    uint32_t* sums = nullptr;
    uint64_t* base = nullptr;
    uint32_t* acc[3] = {nullptr, nullptr, nullptr};
    uint16_t* cnt[3] = {nullptr, nullptr, nullptr};
    hipEvent_t copied = nullptr, computed = nullptr, drained = nullptr;
};

void free_buffers(Slot& s) {
    for (void* p : {(void*)s.rd, (void*)s.rf, (void*)s.len, (void*)s.E, (void*)s.off, (void*)s.sums, (void*)s.base})
        if (p) (void)hipFree(p);
    for (int f = 0; f < 3; ++f) {
        if (s.acc[f]) (void)hipFree(s.acc[f]);
        if (s.cnt[f]) (void)hipFree(s.cnt[f]);
        s.acc[f] = nullptr;
        s.cnt[f] = nullptr;
    }
    s.rd = s.rf = s.off = s.base = nullptr;
    s.len = nullptr;
    s.E = nullptr;
    s.sums = nullptr;
}

}  // namespace

// What a context keeps between streamed batches: two slots of device buffers,
// the three streams and their events, which were made for each call before.
// Buffers above kStreamKeepBytes are given back when the call ends, everything
// when the context is destroyed.  Nothing of a batch is kept: a call ends with
// its streams idle.
namespace paf {
struct StreamWs {
    Slot slots[2];
    hipStream_t in = nullptr, comp = nullptr, out = nullptr;
    uint64_t words = 0, pairs = 0;   // a slot's capacity
    uint32_t filters = 0;            // ... and the stages it has outputs for
    size_t bytes = 0;
};

void stream_ws_free(StreamWs* w) {
    if (!w) return;
    for (auto& s : w->slots) {
        free_buffers(s);
        for (hipEvent_t e : {s.copied, s.computed, s.drained})
            if (e) (void)hipEventDestroy(e);
    }
    for (hipStream_t st : {w->in, w->comp, w->out})
        if (st) (void)hipStreamDestroy(st);
    delete w;
}
}  // namespace paf

namespace {

constexpr size_t kStreamKeepBytes = (size_t)2 << 30;

// Bytes of both slots for chunks of `pairs` pairs and `words` words per array.
size_t slots_bytes(uint64_t words, uint64_t pairs, uint32_t filters) {
    const uint64_t nsb = (pairs + kScanBlock - 1) / kScanBlock;
    const uint64_t stages = (uint64_t)__builtin_popcount(filters);
    return 2 * (words * 16 + pairs * 11 + nsb * 12 + stages * (pairs / 8 + pairs * 2));
}

// The slots' buffers made anew; false (and none) if the memory does not suffice.
bool make_slots(StreamWs* w, uint64_t words, uint64_t pairs, uint32_t filters) {
    for (auto& s : w->slots) free_buffers(s);
    w->words = w->pairs = 0;
    w->filters = 0;
    w->bytes = 0;
    const uint64_t nsb = (pairs + kScanBlock - 1) / kScanBlock;
    for (auto& s : w->slots) {
        bool ok = hipMalloc(&s.rd, words * 8) == hipSuccess && hipMalloc(&s.rf, words * 8) == hipSuccess &&
                  hipMalloc(&s.len, pairs * 2) == hipSuccess && hipMalloc(&s.E, pairs) == hipSuccess &&
                  hipMalloc(&s.off, pairs * 8) == hipSuccess && hipMalloc(&s.sums, nsb * 4) == hipSuccess &&
                  hipMalloc(&s.base, nsb * 8) == hipSuccess;
        for (int f = 0; f < 3 && ok; ++f)
            if ((filters >> f) & 1u)
                ok = hipMalloc(&s.acc[f], pairs / 8) == hipSuccess && hipMalloc(&s.cnt[f], pairs * 2) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            for (auto& t : w->slots) free_buffers(t);
            return false;
        }
    }
    w->words = words;
    w->pairs = pairs;
    w->filters = filters;
    w->bytes = slots_bytes(words, pairs, filters);
    return true;
}

// Slots for chunks of `pairs` pairs and `words` words per array: the kept ones,
// or new ones that fit the earlier shapes too while those can be kept, or just
// this call's.
paf_status ensure_stream_ws(paf_ctx* ctx, uint64_t words, uint64_t pairs, uint32_t filters) {
    StreamWs* w = ctx->stream_ws;
    if (!w) {
        w = new (std::nothrow) StreamWs();
        if (!w) return fail(PAF_ERR_NOMEM, "host allocation failed");
        ctx->stream_ws = w;
        bool ok = true;
        for (hipStream_t* st : {&w->in, &w->comp, &w->out})
            ok = ok && hipStreamCreateWithFlags(st, hipStreamNonBlocking) == hipSuccess;
        for (auto& s : w->slots)
            for (hipEvent_t* e : {&s.copied, &s.computed, &s.drained})
                ok = ok && hipEventCreateWithFlags(e, hipEventDisableTiming) == hipSuccess;
        if (!ok) {
            stream_ws_free(w);
            ctx->stream_ws = nullptr;
            return fail(PAF_ERR_DEVICE, "streams and events");
        }
    }
    if (w->words >= words && w->pairs >= pairs && (w->filters & filters) == filters) return PAF_OK;
    const uint64_t all_words = std::max(words, w->words), all_pairs = std::max(pairs, w->pairs);
    const uint32_t all_filters = filters | w->filters;
    if (slots_bytes(all_words, all_pairs, all_filters) <= kStreamKeepBytes && make_slots(w, all_words, all_pairs, all_filters))
        return PAF_OK;
    return make_slots(w, words, pairs, filters) ? PAF_OK : fail(PAF_ERR_NOMEM, "streaming buffers");
}

// Words of pairs [a, b), or UINT64_MAX when a length is outside [1, max_len]
// (two reductions without a branch, so the loop runs on vectors).
uint64_t count_words(const uint16_t* len, uint64_t a, uint64_t b, uint32_t max_len) {
    uint64_t total = 0;
    uint16_t most = 0, least = UINT16_MAX;
    while (a < b) {
        const uint64_t e = std::min(b, a + 65536);
        uint32_t w = 0;
        for (uint64_t p = a; p < e; ++p) {
            const uint16_t l = len[p];
            most = std::max(most, l);
            least = std::min(least, l);
            w += ((uint32_t)l + 31u) >> 5;
        }
        total += w;
        a = e;
    }
    return least < 1 || most > max_len ? UINT64_MAX : total;
}

}  // namespace

extern "C" {

paf_status paf_stream_filter(paf_ctx* ctx, const paf_host_batch* hb, uint64_t chunk_pairs, uint32_t filters,
                             int learned, const paf_out* host_out, paf_stream_stats* stats) {
    if (!ctx || !hb || !host_out) return fail(PAF_ERR_ARG, "ctx/batch/out is NULL");
    if (!hb->reads || !hb->refs || !hb->len || !hb->E) return fail(PAF_ERR_ARG, "host batch has a NULL array");
    if (hb->n_pairs == 0) return fail(PAF_ERR_ARG, "batch has no pairs");
    if (chunk_pairs == 0 || chunk_pairs % 64 != 0) return fail(PAF_ERR_ARG, "chunk_pairs must be a positive multiple of 64");
    if (filters == 0 || filters > 7u) return fail(PAF_ERR_ARG, "filters must be a nonzero mask of PAF_* bits");
    if (hb->max_len < 1 || hb->max_len > PAF_MAX_LEN || hb->max_E > PAF_MAX_E)
        return fail(PAF_ERR_RANGE, "max_len/max_E outside the supported range");
    for (int f = 0; f < 3; ++f)
        if ((filters >> f) & 1u)
            if (!host_out->accept_bits[f] || !host_out->count[f])
                return fail(PAF_ERR_ARG, "a requested filter has a NULL output pointer");
    if (learned && !ctx->mlp_ready) return fail(PAF_ERR_STATE, "no cost model: call paf_mlp_set_params first");
    PAF_HIP(hipSetDevice(ctx->device), "hipSetDevice");

    const uint64_t n = hb->n_pairs;
    const uint64_t nchunks = (n + chunk_pairs - 1) / chunk_pairs;
    // Word position of every chunk's first pair (pairs are stored back to
    // back), counted and range-checked by one thread per quarter million pairs
    // (16 at most) before anything is copied.
    std::vector<uint64_t> cw;
    try {
        cw.assign(nchunks + 1, 0);
        const uint64_t T = std::min<uint64_t>(std::min<uint64_t>(16, nchunks), std::max<uint64_t>(1, n >> 18));
        auto count = [&](uint64_t t) {
            for (uint64_t c = t; c < nchunks; c += T)
                cw[c + 1] = count_words(hb->len, c * chunk_pairs, std::min(n, (c + 1) * chunk_pairs), hb->max_len);
        };
        std::vector<std::thread> pool;
        uint64_t t = 1;
        try {
            pool.reserve(T);
            for (; t < T; ++t) pool.emplace_back(count, t);
        } catch (...) {
            // Fewer threads than wanted: this one counts the rest.
        }
        count(0);
        for (; t < T; ++t) count(t);
        for (auto& th : pool) th.join();
    } catch (...) {
        return fail(PAF_ERR_NOMEM, "host allocation failed");
    }
    uint64_t max_words = 0;
    for (uint64_t c = 0; c < nchunks; ++c) {
        if (cw[c + 1] == UINT64_MAX) return fail(PAF_ERR_RANGE, "a pair length is outside [1, max_len]");
        max_words = std::max(max_words, cw[c + 1]);
        cw[c + 1] += cw[c];
    }
    // (slots no larger than the batch: outputs come in words of 32 pairs)
    const uint64_t slot_pairs = std::min(chunk_pairs, (n + 63) / 64 * 64);
    paf_status st = ensure_stream_ws(ctx, max_words, slot_pairs, filters);
    if (st != PAF_OK) return st;
    StreamWs& ws = *ctx->stream_ws;

    // Chunk c is copied in on one stream, filtered on the second and its
    // results copied out on the third, each as soon as the slot's chunk c - 2
    // has left that stage: the next chunk's words come in while this one is
    // filtered.  (With the results on the stream of the incoming copies, every
    // chunk's copy waited for the previous chunk's filter.)  2M pairs in chunks
    // of 512k: 5.53 ms with two streams, 4.08 on a new context, 3.79 from its
    // second call on, whose buffers are there: 50 of the link's 57 GB/s.
    double h2d = 0;
    const auto t0 = std::chrono::steady_clock::now();
    for (uint64_t c = 0; c < nchunks && st == PAF_OK; ++c) {
        Slot& s = ws.slots[c % 2];
        const uint64_t a = c * chunk_pairs, m = std::min(chunk_pairs, n - a);
        const uint64_t w0 = cw[c], nw = cw[c + 1] - cw[c];
        bool ok = c < 2 || hipStreamWaitEvent(ws.in, s.computed, 0) == hipSuccess;
        ok = ok && hipMemcpyAsync(s.rd, hb->reads + w0, nw * 8, hipMemcpyHostToDevice, ws.in) == hipSuccess &&
             hipMemcpyAsync(s.rf, hb->refs + w0, nw * 8, hipMemcpyHostToDevice, ws.in) == hipSuccess &&
             hipMemcpyAsync(s.len, hb->len + a, m * 2, hipMemcpyHostToDevice, ws.in) == hipSuccess &&
             hipMemcpyAsync(s.E, hb->E + a, m, hipMemcpyHostToDevice, ws.in) == hipSuccess &&
             hipEventRecord(s.copied, ws.in) == hipSuccess && hipStreamWaitEvent(ws.comp, s.copied, 0) == hipSuccess &&
             (c < 2 || hipStreamWaitEvent(ws.comp, s.drained, 0) == hipSuccess);
        if (!ok) { st = fail(PAF_ERR_DEVICE, "chunk copy"); break; }
        h2d += (double)nw * 16 + (double)m * 3;
        const uint32_t nb = (uint32_t)((m + kScanBlock - 1) / kScanBlock);
        hipLaunchKernelGGL(words_block_sum_kernel, dim3(nb), dim3(256), 0, ws.comp, s.len, m, s.sums);
        hipLaunchKernelGGL(block_base_kernel, dim3(1), dim3(1024), 0, ws.comp, s.sums, nb, s.base);
        hipLaunchKernelGGL(words_offset_kernel, dim3(nb), dim3(kScanBlock), 0, ws.comp, s.len, m, s.base, s.off);
        paf_batch b{};
        b.reads = s.rd;
        b.refs = s.rf;
        b.word_offset = s.off;
        b.len = s.len;
        b.E = s.E;
        b.max_len = hb->max_len;
        b.max_E = hb->max_E;
        b.n_pairs = m;
        paf_out o{};
        for (int f = 0; f < 3; ++f) {
            o.accept_bits[f] = s.acc[f];
            o.count[f] = s.cnt[f];
        }
        st = !learned ? paf_filter(ctx, &b, filters, &o, ws.comp)
             : filters == PAF_SNEAKYSNAKE ? paf_filter_bucketed_local(ctx, &b, &o, ws.comp)
                                          : paf_filter_bucketed(ctx, &b, filters, &o, ws.comp);
        if (st != PAF_OK) break;
        ok = hipEventRecord(s.computed, ws.comp) == hipSuccess && hipStreamWaitEvent(ws.out, s.computed, 0) == hipSuccess;
        for (int f = 0; f < 3 && ok; ++f)
            if ((filters >> f) & 1u)
                ok = hipMemcpyAsync(host_out->accept_bits[f] + a / 32, s.acc[f], (m + 31) / 32 * 4,
                                    hipMemcpyDeviceToHost, ws.out) == hipSuccess &&
                     hipMemcpyAsync(host_out->count[f] + a, s.cnt[f], m * 2, hipMemcpyDeviceToHost, ws.out) ==
                         hipSuccess;
        ok = ok && hipEventRecord(s.drained, ws.out) == hipSuccess;
        if (!ok) st = fail(PAF_ERR_DEVICE, "chunk results");
    }
    for (hipStream_t x : {ws.in, ws.comp, ws.out})
        if (hipStreamSynchronize(x) != hipSuccess && st == PAF_OK) st = fail(PAF_ERR_DEVICE, "stream synchronisation");
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (ws.bytes > kStreamKeepBytes) {
        for (auto& s : ws.slots) free_buffers(s);
        ws.words = ws.pairs = 0;
        ws.filters = 0;
        ws.bytes = 0;
    }
    if (st != PAF_OK) return st;
    if (stats) {
        stats->seconds = secs;
        stats->h2d_bytes = h2d;
        stats->chunks = nchunks;
    }
    return PAF_OK;
}

}  // extern "C"
